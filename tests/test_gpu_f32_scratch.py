"""fp32 calls of one shard on matrices of one column or one row, with K slices: right results, and nothing written behind the
workspace that vp_workspace_bytes asks for."""
import pytest
import torch

pytestmark = pytest.mark.gpu

GUARD = 1 << 18


@pytest.mark.parametrize("N,h,Vs", [(4096, 4096, 1), (2048, 1024, 1), (8192, 64, 1), (5000, 1, 192), (64, 1, 128), (1, 1, 8192),
                                    (8192, 1, 1), (1, 64, 4096)])
def test_nothing_is_written_behind_the_workspace(N, h, Vs):
    import paper_2411_05288_amd as vp
    B = vp.binding
    print("scratch", N, h, Vs, flush=True)
    g = torch.Generator(device="cuda").manual_seed(N + h + Vs)
    H = torch.randn((N, h), generator=g, device="cuda")
    W = torch.randn((Vs, h), generator=g, device="cuda") * (0.1 if h > 1 else 0.5)
    labels = torch.randint(-1, Vs + 1, (N,), generator=g, device="cuda")
    f = dict(device="cuda", dtype=torch.float32)
    lmax, lsum, ltgt, A = torch.empty(N, **f), torch.empty(N, **f), torch.empty(N, **f), torch.empty(N, h, **f)
    Bm, dH, dW = torch.empty(N, h, **f), torch.empty(N, h, **f), torch.empty(Vs, h, **f)

    def workspace(call):
        n = vp.vp_workspace_bytes(call, N, h, Vs, vp.VP_F32, 0)
        whole = torch.full((n + GUARD,), 0xA5, dtype=torch.uint8, device="cuda")
        return whole, whole[:n]

    whole, ws = workspace(B.VP_CALL_OUTPUT_FWD_ALG2)
    vp.vp_output_fwd_alg2(H, W, labels, 0, lmax, lsum, ltgt, A, Bm, None, ws)
    torch.cuda.synchronize()
    assert bool((whole[ws.numel():] == 0xA5).all())
    Hd, Wd = H.double(), W.double()
    Y = Hd @ Wd.t()
    P = torch.softmax(Y, 1)
    # a sum is rounded at most 6 times per 16 k and once per slice, each time by 2^-23 of a partial sum; softmax inherits the
    # logits' and statistics' errors (< 2^-17)
    bar = lambda K: (6 * (K / 16 + 1) + 64) * 2.0 ** -23
    assert bool(((A.double() - P @ Wd).abs() <= (bar(Vs) + 2.0 ** -17) * (P @ Wd.abs())).all())

    whole, ws = workspace(B.VP_CALL_OUTPUT_BWD)
    vp.vp_output_bwd(H, W, labels, 0, lmax, lsum, None, 1.0 / N, dH, dW, ws, dh_overwrite=True)
    torch.cuda.synchronize()
    assert bool((whole[ws.numel():] == 0xA5).all())
    D = ws[:N * Vs * 4].view(torch.float32).view(N, Vs).double()     # D as the call formed it, dense
    own = (labels >= 0) & (labels < Vs)
    want = P.clone()
    want[own, labels[own]] -= 1.0
    assert bool(((D - want / N).abs() <= 2.0 ** -17 / N).all())
    assert bool(((dH.double() - D @ Wd).abs() <= bar(Vs) * (D.abs() @ Wd.abs())).all())
    assert bool(((dW.double() - D.t() @ Hd).abs() <= bar(N) * (D.abs().t() @ Hd.abs())).all())
