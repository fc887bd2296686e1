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
