"""Pass S and the barrier of Algorithm 2 with all shards of the device in one call, against shard by shard."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def plans(N, h, rows, dtype, save_logits, vocab_size=None, seed=3):
    import paper_2411_05288_amd as vp
    g = torch.Generator(device="cuda").manual_seed(seed)
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    H = torch.randn((N, h), generator=g, device="cuda").to(t)
    W = [(torch.randn((n, h), generator=g, device="cuda") * 0.1).to(t) for n in rows]
    labels = torch.randint(0, vocab_size or sum(rows), (N,), generator=g, device="cuda")
    labels[::7] = sum(rows) + 5           # nobody's
    labels[1::11] = -1
    B = vp.binding
    size, out = B.vp_output_group_workspace_bytes, []

    def refuse(which, *a):
        if which == B.VP_CALL_OUTPUT_FWD_ALG2:
            raise B.VPError("one by one")
        return size(which, *a)

    for f in (size, refuse):
        B.vp_output_group_workspace_bytes = f
        try:
            p = vp.OutputLayerPlan(H, W, labels, save_logits, vocab_size=vocab_size, algorithm=2)
        finally:
            B.vp_output_group_workspace_bytes = size
        p.workspace.fill_(0xFF)
        p.dH.fill_(float("nan"))
        p.step()
        torch.cuda.synchronize()
        out.append(p)
    return out


def check(one, each, dtype):
    assert one.grouped_S and not each.grouped_S
    # the per-shard fp32 products may cut K elsewhere: statistics, logits and dW to an fp32 sum of at most 2048 terms
    for name in ("local_max", "local_sumexp", "local_target", "global_max", "global_sumexp", "loss_rows"):
        a, b = getattr(one, name), getattr(each, name)
        assert torch.equal(a, b) if dtype == "bf16" else torch.allclose(a, b, rtol=1e-5, atol=1e-5), name
    for a, b in zip(one.dW, each.dW):
        assert torch.equal(a, b) if dtype == "bf16" else torch.allclose(a, b, rtol=1e-4, atol=1e-7)
    for r in range(one.live):
        assert torch.equal(one.Bm[r], each.Bm[r])
    # the same softmax values (fp32: 2^-17 apart for logits and statistics that are off by 4 ulp), summed in another order where
    # K is cut into slices: at most 17 * 64 fp32 additions
    V = one.vocab_size
    W = torch.cat(one.W).double()[:V]
    P = torch.softmax(one.H.double() @ W.t(), 1)
    mag = P @ W.abs()
    eps = 1100 * 2.0 ** -24 if dtype == "bf16" else 2.0 ** -16
    for r in range(one.live):
        w = one.W[r].double()[:one.valid[r]].abs()
        p_r = P[:, one.offsets[r]:one.offsets[r] + one.valid[r]]
        bar = 1.1 * eps * (p_r / p_r.sum(1, keepdim=True)) @ w + 1e-12
        assert bool(((one.A[r] - each.A[r]).abs() <= bar).all()), r
    assert bool(((one.dH - each.dH).abs() <= (1.1 * eps * mag + 2.0 ** -22 * W.abs().max()) * one.grad_scale).all())


@pytest.mark.parametrize("dtype,save_logits", [("bf16", True), ("bf16", False), ("f32", True), ("f32", False)])
@pytest.mark.parametrize("N,h,rows,vocab", [
    (70, 72, [300, 131], None),              # ragged tiles, few tokens, odd rows
    (300, 64, [513, 513, 513], 1301),        # padding in the last shard
    (33, 37, [66, 70, 5], None),             # rows that are not 16-byte aligned: the generic kernel
    (512, 1024, [1000, 1000], None),         # K slices of A
    (40, 256, [64] * 5, 170),                # shards that are all padding
    (1025, 128, [260] * 16, None),           # more rows than one workgroup combines
])
def test_group_equals_shard_by_shard(N, h, rows, vocab, dtype, save_logits):
    print("alg2 group", N, h, rows, vocab, dtype, save_logits, flush=True)
    check(*plans(N, h, rows, dtype, save_logits, vocab), dtype)


@pytest.mark.parametrize("N,h,rows,vocab", [(70, 256, [4000, 4000, 40], None), (600, 256, [9000, 9000, 64], None),
                                            (40, 1024, [3000] * 4, 9001)])
def test_k_slices_and_a_short_last_shard(N, h, rows, vocab):
    # the longest shard is cut into more K slices than the last one has k tiles: some of its slices are empty
    import paper_2411_05288_amd as vp
    print("alg2 short", N, h, rows, vocab, flush=True)
    one, each = plans(N, h, rows, "bf16", True, vocab)
    B, live = vp.binding, one.valid[:one.live]
    D = sum(N * ((n + 63) // 64 * 64) * 2 for n in live)
    slices = vp.vp_output_group_workspace_bytes(B.VP_CALL_OUTPUT_FWD_ALG2, N, h, live, vp.VP_BF16, B.VP_SAVE_LOGITS) - D
    assert slices // (len(live) * N * h * 4) > (live[-1] + 63) // 64
    check(one, each, "bf16")


def test_group_with_the_generic_kernel():
    import paper_2411_05288_amd as vp
    lib = vp.binding.load_library()
    lib.vp_profile_force_generic_gemm(1)
    try:
        check(*plans(300, 64, [513, 300], "bf16", True), "bf16")
    finally:
        lib.vp_profile_force_generic_gemm(0)


def test_more_shards_than_one_call_takes():
    import paper_2411_05288_amd as vp
    one, each = plans(64, 64, [70] * 17, "bf16", True)
    assert not one.grouped_S and one.grouped
    assert torch.equal(one.dH, each.dH)
    with pytest.raises(vp.VPError):
        vp.vp_output_group_workspace_bytes(vp.binding.VP_CALL_OUTPUT_FWD_ALG2, 64, 64, [70] * 17, vp.VP_BF16, 0)
