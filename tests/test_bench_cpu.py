"""The figures bench.py attaches to a launch belong to the same launch: counters copied from a profile of launches that
serve all shards are not quoted for launches of one shard, nor the reverse."""
import pytest

import bench
import synth_inputs as si


def output_bytes(cfg, kernel):
    if isinstance(cfg, si.EmbedConfig):
        return cfg.p * cfg.N * cfg.h * 2
    return {"gemm_bf16_fwd_stats": 2 * cfg.N * cfg.V * bool(cfg.save_logits), "gemm_bf16_dlogits": 2 * cfg.N * cfg.V,
            "gemm_bf16_dH": 4 * cfg.N * cfg.h, "gemm_bf16_dW": 4 * cfg.V * cfg.h}[kernel]


@pytest.mark.parametrize("name", sorted(bench.PMC_KIB))
def test_counter_traffic_covers_what_a_launch_of_all_shards_writes(name):
    cfg = si.CONFIGS[name]
    for kernel in bench.PMC_KIB[name]:
        assert bench.pmc_traffic(name, kernel, 1.0) >= output_bytes(cfg, kernel), kernel
        assert bench.pmc_traffic(name, kernel, float(cfg.p)) is None


@pytest.mark.parametrize("launches", [1, 16])
def test_gemm_roofline_per_launch_figures_agree(launches):
    cfg = si.CONFIGS["cfg4_very_large_vocab"]
    k = {"gemm_bf16_dW": {"ms_per_launch": 14.0 / launches, "launches_per_step": float(launches), "ms_per_step": 14.0}}
    r = bench.gemm_roofline(cfg, k)
    flops = 2.0 * cfg.N * cfg.h * cfg.V
    assert r["flops_per_launch"] * launches == pytest.approx(flops)
    assert r["achieved"] == pytest.approx(flops / 14e-3 / 1e12)
    assert (r["traffic"] is None) == (launches != 1)
    if launches == 1:
        assert r["traffic"] > r["algorithmic_bytes_per_launch"]
