"""The scatter-add of few tokens (no sort): around 64 tokens per ballot, the largest token count and product of tokens and column
slabs, rows of one to all tokens, several long rows in one workgroup, against the in-order fp32 loop bit for bit."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def ids_of(kind, N, V, rng):
    if kind == "uniform":
        return rng.integers(0, V, N)
    if kind == "one":
        return np.full(N, V - 1)
    if kind == "few":                     # rows of more than 64 tokens from 200 tokens on
        return rng.integers(0, 3, N) * (V // 3)
    ids = rng.integers(0, V, N)           # "mixed": a long row, ids that nobody has, rows of 5 to 30 tokens
    ids[rng.random(N) < 0.4] = 1
    ids[rng.random(N) < 0.2] = rng.integers(0, 4) + 2
    ids[::9] = V + 7
    ids[1::17] = -3
    return ids


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("kind", ["uniform", "one", "few", "mixed"])
@pytest.mark.parametrize("N,h,p", [(1, 8, 1), (63, 130, 3), (64, 129, 2), (65, 64, 1), (200, 257, 2), (511, 40, 3), (512, 2048, 2),
                                   (512, 1024, 1), (513, 64, 2), (256, 4096, 1), (257, 4096, 1), (128, 8192, 2)])
def test_few_tokens_sum_in_token_order(N, h, p, kind, dtype):
    import paper_2411_05288_amd as vp
    Vs = 40
    rng = np.random.default_rng(100 * N + h)
    ids = ids_of(kind, N, p * Vs, rng)
    print("few tokens", N, h, p, kind, dtype, flush=True)
    g = torch.from_numpy(rng.standard_normal((N, h)).astype(np.float32)).to(dtype)
    start = rng.standard_normal((p * Vs, h)).astype(np.float32)
    d = [torch.from_numpy(start[r * Vs:(r + 1) * Vs].copy()).cuda() for r in range(p)]
    vp.embedding_backward(g.cuda(), torch.from_numpy(ids.astype(np.int64)).cuda(), Vs, p, d)
    torch.cuda.synchronize()
    ref, gf = start.copy(), g.float().numpy()
    for t, i in enumerate(ids):
        if 0 <= i < p * Vs:
            ref[i] += gf[t]
    got = np.concatenate([x.cpu().numpy() for x in d])
    assert np.array_equal(got.view(np.uint32), ref.view(np.uint32))
