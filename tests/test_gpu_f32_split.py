"""fp32 products from bf16 parts: precision of an fp32 sum, the whole range of exponents, infinities where fp32 has them."""
import pytest
import torch

pytestmark = pytest.mark.gpu

# (N, h, rows per shard): tiles of 64 x 64 (with K slices of dH), 128 x 128, 256 x 128; remainders in every direction, rows
# that are not 16-byte aligned
SHAPES = [(70, 72, [300, 131]), (33, 257, [129]), (300, 200, [2500, 2400]), (601, 1100, [2053, 2049]), (520, 68, [9000, 8001])]


def plan_of(N, h, rows, seed, grad_scale=None):
    import paper_2411_05288_amd as vp
    g = torch.Generator(device="cuda").manual_seed(seed)
    H = torch.randn((N, h), generator=g, device="cuda")
    W = [torch.randn((n, h), generator=g, device="cuda") * 0.05 for n in rows]
    labels = torch.randint(0, sum(rows), (N,), generator=g, device="cuda")
    plan = vp.OutputLayerPlan(H, W, labels, True, grad_scale)
    plan.workspace.fill_(0xFF)
    return plan


def step(plan):
    plan.step()
    torch.cuda.synchronize()
    return plan


@pytest.mark.parametrize("N,h,rows", SHAPES)
def test_products_have_the_error_of_an_fp32_sum(N, h, rows):
    print("split", N, h, rows, flush=True)
    plan = step(plan_of(N, h, rows, 5))
    H, W = plan.H.double(), torch.cat(plan.W).double()
    Y = H @ W.t()
    D = torch.softmax(Y, 1)
    D[torch.arange(N, device="cuda"), plan.labels] -= 1.0
    D /= N

    def check(got, A, B, D_error):
        # a sum is rounded at most 6 times per 16 k, each time by 2^-23 of a partial sum, itself at most sum |a b|; a random
        # walk of them for the 2-norm.  D_error: relative error of the elements of D that the kernel formed (fp32 statistics and
        # logits), which its products inherit.
        ref, mag = A @ B, A.abs() @ B.abs()
        n = 6 * (A.shape[1] / 16 + 1)
        err = (got.double() - ref).abs()
        assert bool((err <= (n * 2.0 ** -23 + D_error) * mag).all())
        assert float(err.norm() / ref.norm()) <= n ** 0.5 * 2.0 ** -23 + D_error

    check(torch.cat(plan.logits, 1), H, W.t(), 0.0)
    # |Y| stays below 16: logits and statistics that are off by 4 ulp of 8..16 move D by 8 ulp, 2^-17 of it
    assert float(Y.abs().max()) < 16
    check(plan.dH, D, W, 2.0 ** -17)
    check(torch.cat(plan.dW), D.t(), H, 2.0 ** -17)


@pytest.mark.parametrize("N,h,rows", SHAPES)
def test_small_gradients_keep_all_bits(N, h, rows):
    # powers of two pass through every product and sum unchanged: the same bits, though softmax * 2^-100 ends in parts far
    # below the smallest bf16
    print("small", N, h, rows, flush=True)
    one, small = step(plan_of(N, h, rows, 6, 1.0)), step(plan_of(N, h, rows, 6, 2.0 ** -100))
    assert torch.equal(small.dH * 2.0 ** 100, one.dH)
    for a, b in zip(small.dW, one.dW):
        assert torch.equal(a * 2.0 ** 100, b)


@pytest.mark.parametrize("N,h,rows", SHAPES)
def test_infinities_and_the_largest_values(N, h, rows):
    print("inf", N, h, rows, flush=True)
    plan = plan_of(N, h, rows, 7)
    clean = torch.cat(step(plan).logits, 1).clone()
    j, k, t = rows[0] - 1, h - 1, N - 1
    plan.W[0][j, k] = float("inf")              # an infinity that fp32 keeps: its column is +-inf by the sign of H
    plan.H[t, 0] = 3.4e38                       # rounds to an infinity in bf16; its row stays finite
    plan.H[t, 1:] = 0.0
    plan.forward()
    torch.cuda.synchronize()
    got = torch.cat(plan.logits, 1)
    others = torch.arange(got.shape[1], device="cuda") != j
    assert torch.equal(got[:t, others], clean[:t, others])
    assert torch.equal(got[:t, j], torch.where(plan.H[:t, k] > 0, float("inf"), float("-inf")))
    want = 3.4e38 * torch.cat(plan.W)[:, 0].double()
    assert bool(((got[t].double() - want).abs() <= 2.0 ** -23 * want.abs())[others].all())


def call_bwd(H, W, labels, Y, grad_scale):
    """vp_output_bwd on given logits with statistics 0 and 1 (D = exp(Y) - one-hot): D as it left it, dH, dW."""
    import paper_2411_05288_amd as vp
    N, h, Vs = H.shape[0], H.shape[1], W.shape[0]
    dH, dW = torch.empty((N, h), device="cuda"), torch.empty((Vs, h), device="cuda")
    n = vp.vp_workspace_bytes(vp.binding.VP_CALL_OUTPUT_BWD, N, h, Vs, vp.VP_F32, vp.VP_SAVE_LOGITS)
    ws = torch.full((n,), 0xFF, dtype=torch.uint8, device="cuda")
    vp.vp_output_bwd(H, W, labels, 0, torch.zeros(N, device="cuda"), torch.ones(N, device="cuda"), Y, grad_scale, dH, dW, ws,
                     dh_overwrite=True)
    torch.cuda.synchronize()
    return ws[:N * Vs * 4].view(torch.float32).view(N, Vs), dH, dW


def call_fwd(H, W):
    import paper_2411_05288_amd as vp
    N, Vs = H.shape[0], W.shape[0]
    out, s = torch.empty((N, Vs), device="cuda"), [torch.empty(N, device="cuda") for _ in range(3)]
    n = vp.vp_workspace_bytes(vp.binding.VP_CALL_OUTPUT_FWD, N, H.shape[1], Vs, vp.VP_F32, vp.VP_SAVE_LOGITS)
    ws = torch.empty((max(n, 256),), dtype=torch.uint8, device="cuda")
    vp.vp_output_fwd(H, W, torch.zeros(N, dtype=torch.int64, device="cuda"), 0, *s, out, ws)
    torch.cuda.synchronize()
    return out


@pytest.mark.parametrize("K", [1, 2, 3, 4])
def test_sums_of_few_products_are_rounded_once_per_product(K):
    # one token, a shard of one row, hidden size 1: no more than the rounding of the K products' sum in fp32
    print("few", K, flush=True)
    g = torch.Generator(device="cuda").manual_seed(K)
    rand = lambda *s: torch.randn(s, generator=g, device="cuda")

    def check(got, A, B):
        A, B = A.double(), B.double()
        assert bool(((got.double() - A @ B).abs() <= K * 2.0 ** -24 * (A.abs() @ B.abs())).all())

    for N, h, Vs in ((K, 70, 131), (70, K, 131), (70, 131, K)):
        H, W = rand(N, h), rand(Vs, h)
        D, dH, dW = call_bwd(H, W, torch.randint(0, Vs, (N,), generator=g, device="cuda"), rand(N, Vs), 1.0)
        if h == K:
            check(call_fwd(H, W), H, W.t())
        if Vs == K:
            check(dH, D, W)
        if N == K:
            check(dW, D.t(), H)


@pytest.mark.parametrize("N,h,rows", SHAPES)
def test_the_smallest_operands_keep_all_bits(N, h, rows):
    # scaling by powers of two leaves every bit alone, also where operands become the smallest numbers that fp32 has
    print("smallest", N, h, rows, flush=True)
    g = torch.Generator(device="cuda").manual_seed(8)
    ints = lambda *s: torch.randint(-2 ** 23, 2 ** 23, s, generator=g, device="cuda").to(torch.float32) * 2.0 ** -23
    Vs = rows[0]
    H, W, labels = ints(N, h), ints(Vs, h), torch.randint(0, Vs, (N,), generator=g, device="cuda")
    Y = torch.randn((N, Vs), generator=g, device="cuda")
    tiny = lambda x: x * 2.0 ** -60 * 2.0 ** -66       # multiples of 2^-149
    for got in (call_fwd(tiny(H), W * 2.0 ** 70), call_fwd(H * 2.0 ** 70, tiny(W))):
        assert torch.equal(got * 2.0 ** 56, call_fwd(H, W))
    _, dH, dW = call_bwd(H, W, labels, Y, 1.0)
    assert torch.equal(call_bwd(H, tiny(W), labels, Y, 2.0 ** 76)[1] * 2.0 ** 50, dH)
    assert torch.equal(call_bwd(tiny(H), W, labels, Y, 2.0 ** 76)[2] * 2.0 ** 50, dW)


def parts(x):
    p0 = x.bfloat16().float()
    p1 = (x - p0).bfloat16().float()
    return p0.double(), p1.double(), (x - p0 - p1).double()


@pytest.mark.parametrize("m,n", [(300, 200), (9000, 2000), (16000, 4096)])      # tiles of 64 x 64, 128 x 128, 256 x 128
@pytest.mark.parametrize("product", ["logits", "dH", "dW"])
def test_every_layout_sums_all_six_part_products(product, m, n):
    # operands just over 1 whose second and third parts are positive and large, so that nothing cancels: leaving out one of the
    # six products of parts shows in every sum.  D = exp(Y) (statistics 0 and 1, labels of nobody), read where the call leaves it.
    print("parts", product, m, n, flush=True)
    K = 48
    g = torch.Generator(device="cuda").manual_seed(m)
    over_one = lambda *s: 1.0 + (torch.randint(192, 255, s, generator=g, device="cuda") * 128 + 60).double() * 2.0 ** -23
    nobody = lambda k: torch.full((k,), -1, dtype=torch.int64, device="cuda")
    if product == "logits":
        A, B = over_one(m, K).float(), over_one(n, K).float()
        got = call_fwd(A, B)
    elif product == "dH":
        W = over_one(K, n).float()
        A, got, _ = call_bwd(torch.zeros(m, n, device="cuda"), W, nobody(m), over_one(m, K).log().float(), 1.0)
        B = W.t()
    else:
        H = over_one(K, n).float()
        D, _, got = call_bwd(H, torch.zeros(m, n, device="cuda"), nobody(K), over_one(K, m).log().float(), 1.0)
        A, B = D.t(), H.t()
    ref = A.double() @ B.double().t()
    # 6 roundings per 16 k and the sum of the two halves of K, each by 2^-23 at most; the products left out, 2^-24 at most
    bar = (6 * (K / 16) + 1) * 2.0 ** -23 + 2.0 ** -24
    assert bool(((got.double() - ref).abs() <= bar * ref).all())
    a, b = parts(A), parts(B)
    for i, j in ((0, 0), (0, 1), (1, 0), (1, 1), (0, 2), (2, 0)):
        assert float((a[i].mean(1).min() * b[j].mean(1).min())) > 2 * bar      # (the test can tell)


@pytest.mark.parametrize("N,h,rows", SHAPES + [(2, 64, [3]), (1000, 1024, [4000])])
def test_non_finite_operands_of_the_gradients(N, h, rows):
    # one infinity in H, one NaN and one value that overflows in W: their columns of dW and dH as fp32 has them, all other
    # elements the same bits as without them
    print("non-finite", N, h, rows, flush=True)
    import paper_2411_05288_amd as vp
    g = torch.Generator(device="cuda").manual_seed(9)
    Vs = rows[0]
    H, W = (torch.randn((n, h), generator=g, device="cuda") for n in (N, Vs))
    Y = torch.randn((N, Vs), generator=g, device="cuda")
    labels = torch.randint(0, Vs, (N,), generator=g, device="cuda")
    D, dH, dW = call_bwd(H, W, labels, Y, 4.0)
    D = D.clone()
    t, j, k = N // 2, Vs - 1, h - 1
    H[t, k] = float("inf")
    W[j, 0], W[0, 1] = float("nan"), 3.4e38
    _, dH1, dW1 = call_bwd(H, W, labels, Y, 4.0)
    assert torch.equal(dW1[:, :k], dW[:, :k]) and torch.equal(dW1[:, k], D[t] * float("inf"))
    assert torch.equal(dH1[:, 2:], dH[:, 2:]) and bool(dH1[:, 0].isnan().all())
    want = 3.4e38 * D[:, 0].double()      # (what W's other rows add is below its last bit)
    finite = want.abs() < 3.4e38
    assert bool(((dH1[:, 1].double() - want).abs() <= 2.0 ** -23 * want.abs())[finite].all())
    assert torch.equal(dH1[~finite, 1], torch.sign(D[~finite, 0]) * float("inf"))
    # added to what is there, once
    n = vp.vp_workspace_bytes(vp.binding.VP_CALL_OUTPUT_BWD, N, h, Vs, vp.VP_F32, vp.VP_SAVE_LOGITS)
    ws, acc = torch.empty((n,), dtype=torch.uint8, device="cuda"), torch.ones((N, h), device="cuda")
    vp.vp_output_bwd(H, W, labels, 0, torch.zeros(N, device="cuda"), torch.ones(N, device="cuda"), Y, 4.0, acc, dW1, ws)
    torch.cuda.synchronize()
    assert torch.equal(acc[:, 1:], dH1[:, 1:] + 1.0) and bool(acc[:, 0].isnan().all())
