"""The fp32 products of one shard write no more scratch than vp_workspace_bytes counts, over sizes that include 1: a matrix of one
column, or of one row, is K-contiguous and K-strided at once, and the K slices of a product must not follow from that."""
import pytest

import paper_2411_05288_amd as vp
from paper_2411_05288_amd import binding as B

SIZES = [1, 2, 3, 63, 64, 65, 100, 128, 135, 192, 257, 1000, 1024, 2048, 4095, 4096, 5000, 8069, 8192]
CALLS = [(B.VP_CALL_OUTPUT_FWD, 1), (B.VP_CALL_OUTPUT_FWD_ALG2, 0), (B.VP_CALL_OUTPUT_BWD, 0)]


@pytest.mark.parametrize("call,flags", CALLS)
def test_scratch_written_is_scratch_counted(call, flags):
    lib = vp.load_library()
    used = 0
    for N in SIZES:
        for h in SIZES:
            for Vs in SIZES:
                # fp32 with the logits kept (forward pass) has no [N, Vs] matrix in the workspace, the others have one
                matrix = 0 if flags else (N * Vs * 4 + 255) // 256 * 256
                written = lib.vp_profile_f32_scratch_written(call, N, h, Vs)
                assert matrix + written <= vp.vp_workspace_bytes(call, N, h, Vs, vp.VP_F32, flags), (N, h, Vs)
                used += written > 0
    assert used > 1000      # (most of these sizes are cut into slices)
