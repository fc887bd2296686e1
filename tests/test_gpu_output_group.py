"""All shards of a device in one call (vp_output_fwd_group / vp_output_bwd_group) against the same shards one by one.

The products of a group run over tiles of all shards, dH over the k tiles of all shards, cut into slices where its output
has few tiles; the shapes sit at the edges of that: shards of unequal size, of less than a tile, of no multiple of
anything; more shards than a launch takes; K slices that begin and end inside shards; the generic kernel's shapes.
"""
import numpy as np
import pytest
import torch

import synth_inputs as si
from gpu_util import to_dev

pytestmark = pytest.mark.gpu

GUARD = 1024


def guarded(shape, dtype):
    n = int(np.prod(shape))
    big = torch.full((n + 2 * GUARD,), 7.0, dtype=dtype, device="cuda")
    return big, big[GUARD:GUARD + n].view(*shape)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("save_logits", [True, False])
@pytest.mark.parametrize("N,h,rows", [
    (64, 128, [256, 256]),                    # one tile row, whole tiles
    (300, 128, [1000, 1000, 936]),            # ragged in every direction, last shard shorter
    (257, 64, [255, 1, 64, 513, 2]),          # shards of less than a tile, odd row counts (rows of the logits unaligned)
    (130, 192, [700] * 19),                   # more shards than a launch takes; many k tiles per output tile: K slices
    (513, 512, [1301, 1299]),                 # K slices that start and end inside a shard
    (200, 72, [500, 500]),                    # h % 64 != 0: masked k tail of the logits product
    (70, 8, [300, 5]), (70, 32, [300, 6]), (300, 40, [512, 260]), (64, 376, [300, 300]),    # k tails of either half
    (65, 30, [77, 130]),                      # rows not 16-byte aligned
    (63, 320, [300, 258]), (65, 320, [300, 258]), (64, 1000, [300] * 5), (1, 64, [256, 7]),    # at most 64 tokens and one more
    (4400, 64, [4400, 300]),                  # more than 16 tile rows
])
def test_group_equals_single_shards(N, h, rows, save_logits, dtype):
    import paper_2411_05288_amd as vp
    p, V = len(rows), sum(rows)
    print("output group", (N, h, rows, save_logits, dtype), flush=True)
    offs = [int(x) for x in np.cumsum([0] + rows[:-1])]
    H = to_dev(si.normal((N, h), 1.0, dtype, 31, si.STREAM_TABLE, 99))
    W = [to_dev(si.normal((n, h), 0.05, dtype, 31, si.STREAM_TABLE, r)) for r, n in enumerate(rows)]
    labels = si.zipf_ids(N, V, 1.1, 31)
    labels[::9] = V + 3                       # owned by no shard
    labels = to_dev(labels)
    f32, dt, code = torch.float32, H.dtype, vp.VP_F32 if dtype == "f32" else vp.VP_BF16
    flags = vp.VP_SAVE_LOGITS if save_logits else 0
    scale = 1.0 / N

    def run(group):
        keep, out = [], {}
        for name, shp, t in [("lm", (p, N), f32), ("ls", (p, N), f32), ("lt", (p, N), f32), ("dH", (N, h), f32)] + \
                [("dW%d" % r, (n, h), f32) for r, n in enumerate(rows)] + \
                [("y%d" % r, (N, n), dt) for r, n in enumerate(rows) if save_logits]:
            big, out[name] = guarded(shp, t)
            keep.append((name, big))
        ys = [out["y%d" % r] for r in range(p)] if save_logits else None
        dWs = [out["dW%d" % r] for r in range(p)]
        gm, gs, lr, lo = (torch.empty((N,), device="cuda") for _ in range(4))
        B = vp.binding
        if group:
            need = max(vp.vp_output_group_workspace_bytes(c, N, h, rows, code, flags) for c in (B.VP_CALL_OUTPUT_FWD, B.VP_CALL_OUTPUT_BWD))
        else:
            need = max(vp.vp_workspace_bytes(c, N, h, n, code, flags) for c in (B.VP_CALL_OUTPUT_FWD, B.VP_CALL_OUTPUT_BWD) for n in rows)
        need = max(need, 256)
        wsb = torch.full((need + 4096,), 0xFF, dtype=torch.uint8, device="cuda")
        ws = wsb[:need]
        if group:
            vp.vp_output_fwd_group(H, W, labels, offs, out["lm"], out["ls"], out["lt"], ys, ws)
        else:
            for r in range(p):
                vp.vp_output_fwd(H, W[r], labels, offs[r], out["lm"][r], out["ls"][r], out["lt"][r], ys[r] if ys else None, ws)
        vp.vp_combine_stats(out["lm"], out["ls"], out["lt"], gm, gs, lr, lo[:1])
        ws.fill_(0xFF)
        results = []
        for over in (True, False):            # overwrite, then add to what is there
            if group:
                vp.vp_output_bwd_group(H, W, labels, offs, gm, gs, ys, scale, out["dH"], dWs, ws, dh_overwrite=over)
            else:
                for r in range(p):
                    vp.vp_output_bwd(H, W[r], labels, offs[r], gm, gs, ys[r] if ys else None, scale, out["dH"], dWs[r], ws,
                                     dh_overwrite=over and r == 0)
            results.append(out["dH"].clone())
        torch.cuda.synchronize()
        for name, big in keep:
            assert bool((big[:GUARD] == 7.0).all()) and bool((big[-GUARD:] == 7.0).all()), name + ": written outside"
        assert bool((wsb[need:] == 0xFF).all()), "workspace written beyond its size"
        out["dH"], out["dH twice"] = results
        return out

    a, b = run(True), run(False)
    # fp32 sums of V terms in another order: each of the two differs from the exact sum by at most (adds in a chain) * 2^-24
    # of the sum of magnitudes; sqrt(V) * 2^-22 of the largest element covers both many times over.  In fp32 the logits (and
    # with them everything) may differ by a few ulp where the single call cut K, so there it holds for every tensor, with
    # chains of max(V, h, N) terms and |Y| of order 1 in the exponent.
    tol = 2.0 ** -22 * max(V, h, N) ** 0.5
    for name in a:
        x, y = a[name].float(), b[name].float()
        if name.startswith("dH") or dtype == "f32":
            assert float((x - y).abs().max()) <= tol * max(float(y.abs().max()), 1e-30), name
        else:
            assert torch.equal(x, y), name

@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("N,h,p", [(70, 64, 3), (33, 30, 2), (16, 8, 17)])     # vector and element paths; more than one launch
def test_dx_alg2_group_equals_single_calls(N, h, p, dtype):
    import paper_2411_05288_amd as vp
    A = [to_dev(si.normal((N, h), 1.0, "f32", 41, si.STREAM_TABLE, r)) for r in range(p)]
    Bm = [to_dev(si.normal((N, h), 1.0, dtype, 42, si.STREAM_TABLE, r)) for r in range(p)]
    lm = to_dev(si.normal((p, N), 1.0, "f32", 43, si.STREAM_TABLE, 0))
    ls = to_dev(si.normal((p, N), 1.0, "f32", 44, si.STREAM_TABLE, 0)).abs() + 1
    lm[p - 1].fill_(float("-inf"))             # a shard that is all padding
    gm, gs = lm.max(0).values.contiguous(), ls.sum(0).contiguous()
    for over in (True, False):
        x = torch.full((N, h), 3.0, device="cuda")
        y = x.clone()
        vp.vp_output_dx_alg2_group(A, Bm, lm, ls, gm, gs, 0.25, x, dh_overwrite=over)
        for r in range(p):
            vp.vp_output_dx_alg2(A[r], Bm[r], lm[r], ls[r], gm, gs, 0.25, y, dh_overwrite=over and r == 0)
        assert torch.equal(x, y)


@pytest.mark.parametrize("algorithm", [1, 2])
@pytest.mark.parametrize("save_logits", [True, False])
def test_plan_with_a_workspace_limit(save_logits, algorithm):
    # shard by shard, with a short shard and one of padding alone; same numbers as in one call per pass
    import paper_2411_05288_amd as vp
    N, h, p, rows, V = 300, 128, 4, 520, 1300
    H, Ws, labels = si.small_output_case(N, h, rows * p, p, "bf16", seed=71, w_std=0.08)
    H, Ws, labels = to_dev(H), [to_dev(w) for w in Ws], to_dev(labels % V)
    plans = []
    for limit in (None, 0):
        plans.append(vp.OutputLayerPlan(H, Ws, labels, save_logits, vocab_size=V, algorithm=algorithm, workspace_limit=limit))
        plans[-1].workspace.fill_(0xFF)
        plans[-1].step()
    torch.cuda.synchronize()
    a, b = plans
    assert a.grouped and not b.grouped and b.workspace.numel() < a.workspace.numel()
    for name in ("loss", "local_max", "local_sumexp", "local_target", "global_max", "global_sumexp"):
        assert torch.equal(getattr(a, name), getattr(b, name)), name
    for x, y in zip(a.dW, b.dW):
        assert torch.equal(x, y)
    # (orders of the sums: see the bound above)
    assert float((a.dH - b.dH).abs().max()) <= 2.0 ** -22 * V ** 0.5 * float(b.dH.abs().max())


@pytest.mark.parametrize("save_logits", [True, False])
@pytest.mark.parametrize("N,h,rows", [
    (16, 2048, [1000, 999]),                  # logits in 8 slices; rows of Y of no multiple of four, so sums element by element
    (16, 1028, [500, 500]),                   # slices of unequal length, 16-byte sums
    (2048, 64, [125] * 16),                   # dW in 8 slices
    (1030, 37, [70, 65, 1]),                  # dW in slices of an odd K, rows of H not 16-byte aligned
    (20, 1023, [64] * 3), (20, 1024, [64] * 3),     # the last K that is not cut and the first that is
    (64, 4096, [64] * 16),                    # shards of one tile: 256 workgroups with either size of tile
    (200, 1024, [70] * 19),                   # more shards than a launch takes
])
def test_fp32_group_with_k_slices(N, h, rows, save_logits):
    # outputs with few tiles and a long K: the logits and dW of all shards are cut into K slices
    test_group_equals_single_shards(N, h, rows, save_logits, "f32")


def test_every_launch_of_a_step_is_timed():
    # dH in K slices, recomputed logits with rows of D to pad: the sum and the fill are launches of their own
    import paper_2411_05288_amd as vp
    H, Ws, labels = si.small_output_case(300, 512, 2600, 2, "bf16", seed=73, w_std=0.08)
    plan = vp.OutputLayerPlan(to_dev(H), [to_dev(w) for w in Ws], to_dev(labels), False)
    plan.step()
    torch.cuda.synchronize()
    vp.vp_profile_enable(True)
    try:
        plan.step()
        torch.cuda.synchronize()
        launches = {k: n for k, (_, n) in vp.vp_profile_read().items()}
    finally:
        vp.vp_profile_enable(False)
    assert launches == {"gemm_bf16_fwd_stats": 1, "fold_partials": 1, "combine_stats": 1, "gemm_bf16_dlogits": 1,
                        "zero_pad_columns": 1, "gemm_bf16_dH": 1, "sum_slices": 1, "gemm_bf16_dW": 1}


@pytest.mark.parametrize("N,h,rows,dtype", [
    (16384, 64, [65536] * 3, "bf16"),         # 2 GiB of D per shard: parts of two shards and of one
    (16384, 64, [32768] * 3, "f32"),          # the same
    (16384, 2048, [64] * 16, "f32"),          # 2 GiB of partial sums of dH: shard by shard
])
def test_parts_by_bytes(N, h, rows, dtype):
    # dH is overwritten by the first part and added to by the second
    test_group_equals_single_shards(N, h, rows, False, dtype)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("N,h,rows", [
    (70, 72, [300, 131]), (64, 72, [300, 131]), (64, 136, [257, 64]),     # masked k tails, two and four row blocks
    (300, 128, [300, 131]), (40, 37, [66, 70]),
])
def test_infinities_and_nan_stay_where_they_are(N, h, rows, dtype):
    # A token row (or vocabulary row) with infinities and NaN: nothing of it reaches another row's logits, statistics or dH
    # through a tile's overhang, where it would meet a zero.  Without it the same sums in the same order: equal bits.
    import paper_2411_05288_amd as vp
    p, V = len(rows), sum(rows)
    print("non-finite", (N, h, rows, dtype), flush=True)
    H = to_dev(si.normal((N, h), 1.0, dtype, 51, si.STREAM_TABLE, 99))
    W = [to_dev(si.normal((n, h), 0.05, dtype, 51, si.STREAM_TABLE, r)) for r, n in enumerate(rows)]
    labels = to_dev(si.zipf_ids(N, V, 1.1, 51))

    def step(H, W):
        plan = vp.OutputLayerPlan(H, W, labels, True)
        plan.workspace.fill_(0xFF)
        plan.step()
        torch.cuda.synchronize()
        return plan

    clean = step(H, W)
    bad = [0, 5, N - 1]
    H2 = H.clone()
    H2[0, :3] = float("inf")
    H2[5, h // 2] = float("nan")
    H2[N - 1, -1] = float("-inf")
    got = step(H2, W)
    good = torch.ones(N, dtype=torch.bool, device="cuda")
    good[bad] = False
    for name in ("local_max", "local_sumexp", "local_target"):
        assert torch.equal(getattr(got, name)[:, good], getattr(clean, name)[:, good]), name
    for name in ("global_max", "global_sumexp", "loss_rows", "dH"):
        assert torch.equal(getattr(got, name)[good], getattr(clean, name)[good]), name
    for y, y0 in zip(got.logits, clean.logits):
        assert torch.equal(y[good], y0[good])
    assert not bool(torch.isfinite(got.loss_rows[bad]).any())
    # the last vocabulary row of the first shard
    W2 = [w.clone() for w in W]
    W2[0][-1, :2] = float("inf")
    W2[0][-1, -1] = float("nan")
    got = step(H, W2)
    assert torch.equal(got.logits[0][:, :-1], clean.logits[0][:, :-1]) and torch.equal(got.logits[1], clean.logits[1])
    assert bool(torch.isnan(got.logits[0][:, -1]).all())
    for name in ("local_max", "local_sumexp", "local_target"):
        assert torch.equal(getattr(got, name)[1], getattr(clean, name)[1]), name
