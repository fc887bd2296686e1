"""Tiles of 64, 128, 192 and 256 token rows in the bf16 products (logits, D formed again, dH, A of Algorithm 2): token counts
around every tile height, a masked k tail, several tile rows, against the oracle with the bars of the main parity tests."""
import pytest

import synth_inputs as si
from test_gpu_next_rows import check_alg2
from test_gpu_output import check_against_oracle

pytestmark = pytest.mark.gpu

TOKENS = [1, 63, 64, 65, 127, 128, 129, 191, 192, 193, 255, 257, 300, 321, 384, 385]


@pytest.mark.parametrize("save_logits", [True, False])
@pytest.mark.parametrize("h", [192, 200])
@pytest.mark.parametrize("N", TOKENS)
def test_token_counts_around_the_tile_heights(N, h, save_logits):
    H, Ws, labels = si.small_output_case(N, h, 1204, 2, "bf16", seed=1500 + N, w_std=0.08)
    print("row blocks", N, h, save_logits, flush=True)
    check_against_oracle(H, Ws, labels, save_logits, tag=str((N, h, save_logits)))


@pytest.mark.parametrize("N,h", [(100, 1024), (100, 1032), (130, 1032), (192, 1024), (192, 2048), (256, 1024)])
def test_more_tiles_than_the_lowest_height_has_room_for(N, h):
    # 133 tile columns: with 64 rows a second round, so 128 (100 tokens), 192 and 256 rows
    H, Ws, labels = si.small_output_case(N, h, 34000, 2, "bf16", seed=1700 + N, w_std=0.03)
    print("row blocks, many columns", N, h, flush=True)
    for save_logits in (True, False):
        check_against_oracle(H, Ws, labels, save_logits, tag=str((N, h, save_logits)))


@pytest.mark.parametrize("N", [64, 129, 300])
def test_a_of_algorithm2_around_the_tile_heights(N):
    print("row blocks, algorithm 2", N, flush=True)
    check_alg2(N, 192, 1204, 2, "bf16", True, seed=1600 + N)

