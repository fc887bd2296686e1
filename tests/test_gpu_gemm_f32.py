"""The fp32 products on the matrix cores at the edges of their tiles: both tile sizes (128 x 128 from 256 tiles on, else
64 x 64), K tails, rows that are not 16-byte aligned, K slices.  Bars as in the main parity tests (1e-5 * max|tensor|
for gradients, 2e-6 * |Y|max for statistics), which are those of an fp32 contraction in any order."""
import pytest

import synth_inputs as si
from test_gpu_output import check_against_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [
    (2050, 36, 2004),      # pass S in 17 x 16 tiles of 128, K = 36: one full step and a tail of 4
    (2049, 37, 2003),      # the same with rows of H, W and Y that are not 16-byte aligned, K tail of 5
    (2050, 2004, 70),      # dH in 17 x 16 tiles of 128, K = 70
    (70, 2004, 2050),      # dW in 17 x 16 tiles of 128, K = 70
    (65, 33, 129),         # one row / column past a tile of 64, one k past a step of 32
    (1, 31, 4099),         # a single token; dH in K slices with an odd K
])
@pytest.mark.parametrize("save_logits", [True, False])
def test_fp32_products_at_tile_edges(shape, save_logits):
    N, h, Vs = shape
    H, Ws, labels = si.small_output_case(N, h, Vs, 1, "f32", seed=1200 + N, w_std=0.08)
    print("case", shape, save_logits, flush=True)
    check_against_oracle(H, Ws, labels, save_logits, tag=str((shape, save_logits)))


@pytest.mark.parametrize("algorithm", [1, 2])
@pytest.mark.parametrize("N,Vs,p", [(65, 130, 1), (1, 7, 1), (40, 1, 1), (1, 1, 1), (65, 130, 2)])
def test_fp32_hidden_size_one(N, Vs, p, algorithm):
    # h = 1: H and W are K-contiguous and K-strided at once; a shard of one row makes D so as well
    import numpy as np
    import torch
    import paper_2411_05288_amd as vp
    from gpu_util import to_dev, to_host
    from oracle import vp_oracle as oc
    H, Ws, labels = si.small_output_case(N, 1, Vs * p, p, "f32", seed=1300 + N, w_std=0.5)
    print("case h=1", N, Vs, p, algorithm, flush=True)
    plan = vp.OutputLayerPlan(to_dev(H), [to_dev(w) for w in Ws], to_dev(labels), True, algorithm=algorithm)
    plan.workspace.fill_(0xFF)
    plan.step()
    torch.cuda.synchronize()
    ref = oc.output_layer(si.as_f64(H), np.concatenate([si.as_f64(w) for w in Ws]), labels)
    # sums of at most 260 terms, each bounded by max|H| or max|W| over N: 1e-5 of those is the fp32 bar of the other tests
    # (not of max|dH|: with one column the two halves of D may cancel)
    dW = np.concatenate([to_host(w) for w in plan.dW])
    assert np.abs(to_host(plan.dH) - ref["dX"]).max() <= 1e-5 * max(np.abs(w).max() for w in Ws) / N
    assert np.abs(dW - ref["dW"]).max() <= 1e-5 * np.abs(H).max()
    assert abs(float(plan.loss.cpu()[0]) - ref["loss"]) <= 1e-5 * max(abs(ref["loss"]), 1.0)
