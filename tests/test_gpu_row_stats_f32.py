"""fp32 row statistics around the row lengths where the kernel changes its number of values per thread, from rows that start at
any element, against float64 from the kept logits."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [[1, 3], [5, 1023], [1024, 1025], [2047, 2049], [2048, 4], [4095, 4097], [4096, 7], [8191, 8193],
                                  [8192, 4096], [20001, 2]])
def test_row_statistics(rows):
    import paper_2411_05288_amd as vp
    N, h = 37, 8
    print("row stats", rows, flush=True)
    g = torch.Generator(device="cuda").manual_seed(11)
    H = torch.randn((N, h), generator=g, device="cuda")
    W = [torch.randn((n, h), generator=g, device="cuda") for n in rows]
    labels = torch.randint(0, sum(rows), (N,), generator=g, device="cuda")
    labels[0], labels[1], labels[2], labels[3] = 0, rows[0] - 1, rows[0], sum(rows) - 1
    plan = vp.OutputLayerPlan(H, W, labels, True)
    plan.forward()
    torch.cuda.synchronize()
    first = 0
    for r, n in enumerate(rows):
        y = plan.logits[r].double()
        m = y.max(1).values
        assert torch.equal(plan.local_max[r].double(), m)
        s = torch.exp(y - m[:, None]).sum(1)
        # expf of a difference that is rounded once: 2^-23 (|y - m| + 2) of each term, and at most n / 256 + 16 roundings of the sum
        bar = 2.0 ** -23 * (float((m[:, None] - y).max()) + 2 + n / 256 + 16)
        assert bool(((plan.local_sumexp[r].double() - s).abs() <= bar * s).all())
        own = (labels >= first) & (labels < first + n)
        t = torch.where(own, y.gather(1, (labels - first).clamp(0, n - 1)[:, None])[:, 0], 0.0)
        assert torch.equal(plan.local_target[r].double(), t)
        first += n
