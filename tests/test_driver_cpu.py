"""Host-side choices of the driver, on CPU tensors: which entry point a call goes to, and with how much workspace.  The
entry points that would launch kernels are replaced by recorders."""
import weakref

import pytest
import torch

import paper_2411_05288_amd as vp
from paper_2411_05288_amd import binding as B, driver


@pytest.fixture
def embed_calls(monkeypatch):
    calls = []
    monkeypatch.setattr(B, "vp_embed_bwd_group",
                        lambda g, ids, off, dt, ws, stream=None: calls.append(("group", [d.data_ptr() for d in dt], ws.numel())))
    monkeypatch.setattr(B, "vp_embed_bwd",
                        lambda g, ids, off, d, ws, stream=None: calls.append(("one", off, d.data_ptr(), ws.numel())))
    return calls


def grads(p, Vs=6, h=8):
    return [torch.zeros(Vs, h) for _ in range(p)]


def test_embedding_backward_takes_one_call_for_shards_of_their_own(embed_calls):
    g, ids, d = torch.zeros(5, 8), torch.zeros(5, dtype=torch.int64), grads(3)
    assert driver.embedding_backward(g, ids, 6, 3, d) is d
    assert [c[0] for c in embed_calls] == ["group"] and embed_calls[0][1] == [t.data_ptr() for t in d]
    # more gradients than shards: the others are left alone
    embed_calls.clear()
    driver.embedding_backward(g, ids, 6, 2, d)
    assert embed_calls[0][1] == [t.data_ptr() for t in d[:2]]
    # one tensor [p, Vs, h] instead of a list, and shards that touch without overlapping
    embed_calls.clear()
    driver.embedding_backward(g, ids, 6, 3, torch.zeros(3, 6, 8))
    assert [c[0] for c in embed_calls] == ["group"]


def test_embedding_backward_refuses_too_few_gradients(embed_calls):
    # a shard without a gradient must not be passed over in silence
    with pytest.raises(IndexError):
        driver.embedding_backward(torch.zeros(5, 8), torch.zeros(5, dtype=torch.int64), 6, 4, grads(2))
    assert embed_calls == []


def test_embedding_backward_of_no_shards(embed_calls):
    assert driver.embedding_backward(torch.zeros(5, 8), torch.zeros(5, dtype=torch.int64), 6, 0) == []
    assert embed_calls == []


@pytest.mark.parametrize("overlap", ["same", "shifted"])
def test_embedding_backward_of_gradients_that_share_memory_goes_in_order(embed_calls, overlap):
    # one launch would add to the same rows from several workgroups at once
    base = torch.zeros(9, 8)
    d = [base[:6], base[:6]] if overlap == "same" else [base[3:9], base[:6]]
    driver.embedding_backward(torch.zeros(5, 8), torch.zeros(5, dtype=torch.int64), 6, 2, d)
    assert [c[:3] for c in embed_calls] == [("one", 0, d[0].data_ptr()), ("one", 6, d[1].data_ptr())]


def test_embedding_backward_workspace_covers_every_gradient(embed_calls):
    # gradients with more rows than Vs go one by one; above 2^19 - 1 rows a call needs the larger workspace
    N, h, rows = 5000, 8, 2 ** 19
    d = [torch.empty(rows, h), torch.empty(6, h)]
    driver.embedding_backward(torch.zeros(N, h), torch.zeros(N, dtype=torch.int64), 6, 2, d)
    assert [c[0] for c in embed_calls] == ["one", "one"]
    assert embed_calls[0][3] >= vp.vp_workspace_bytes(B.VP_CALL_EMBED_BWD, N, h, rows, vp.VP_F32, 0)


@pytest.mark.parametrize("table,grad", [(torch.bfloat16, torch.float32), (torch.float32, torch.bfloat16)])
def test_embedding_plan_workspace_fits_a_gradient_of_the_other_type(table, grad):
    # at 4 GB of fp32 gradients the scatter-add takes another path than at 2 GB of bf16 ones, with a larger workspace
    N, h = 8192, (1 << 17) + 8
    plan = driver.EmbeddingPlan([torch.empty(2, h, dtype=table)], torch.zeros(N, dtype=torch.int64), None)
    code = vp.VP_F32 if grad == torch.float32 else vp.VP_BF16
    assert plan.workspace.numel() >= vp.vp_workspace_bytes(B.VP_CALL_EMBED_BWD, N, h, 2, code, 0)


def output_plan(algorithm=1, **kw):
    N, h, p, rows = 300, 64, 4, 1000
    return driver.OutputLayerPlan(torch.zeros(N, h, dtype=torch.bfloat16),
                                  [torch.zeros(rows, h, dtype=torch.bfloat16) for _ in range(p)],
                                  torch.zeros(N, dtype=torch.int64), algorithm=algorithm, **kw)


def one_shard_bytes(algorithm):
    fwd = B.VP_CALL_OUTPUT_FWD if algorithm == 1 else B.VP_CALL_OUTPUT_FWD_ALG2
    return max(B.vp_workspace_bytes(c, 300, 64, 1000, vp.VP_BF16, B.VP_SAVE_LOGITS) for c in (fwd, B.VP_CALL_OUTPUT_BWD))


def pass_T_bytes(algorithm):
    return B.vp_output_group_workspace_bytes(B.VP_CALL_OUTPUT_BWD, 300, 64, [1000] * 4, vp.VP_BF16,
                                             B.VP_SAVE_LOGITS | (B.VP_SKIP_DH if algorithm == 2 else 0))


@pytest.mark.parametrize("algorithm", [1, 2])
def test_output_plan_workspace_limit(algorithm):
    full = output_plan(algorithm)
    assert full.grouped and full.workspace.numel() > one_shard_bytes(algorithm)
    assert output_plan(algorithm, workspace_limit=full.workspace.numel()).grouped
    for limit in (pass_T_bytes(algorithm) - 1, 0):
        small = output_plan(algorithm, workspace_limit=limit)
        assert not small.grouped and small.workspace.numel() == one_shard_bytes(algorithm)


def test_algorithm2_plan_with_room_for_pass_T_alone(monkeypatch):
    # pass S of all shards needs more than pass T: without room for it the barrier and pass T still go in one call each
    full, bwd = output_plan(2), pass_T_bytes(2)
    assert full.grouped_S and bwd < full.workspace.numel() and torch.is_tensor(full.A)
    limits = [dict(workspace_limit=full.workspace.numel() - 1), dict(workspace_limit=bwd)]
    for kw in limits:
        small = output_plan(2, **kw)
        assert small.grouped and not small.grouped_S and small.workspace.numel() == bwd and isinstance(small.A, list)
    empty = torch.empty

    def full_device(shape, *a, dtype=None, **kw):
        if dtype == torch.uint8 and shape[0] > bwd:
            raise torch.OutOfMemoryError("no room")
        return empty(shape, *a, dtype=dtype, **kw)

    monkeypatch.setattr(torch, "empty", full_device)
    small = output_plan(2)
    assert small.grouped and not small.grouped_S and small.workspace.numel() == bwd


def test_algorithm2_plan_on_a_device_with_little_room(monkeypatch):
    # A and B of all shards come before the larger workspace: what has room for one shard's workspace next to them still runs
    room, empty = [0], torch.empty

    def small_device(shape, *a, dtype=None, **kw):
        t = empty(shape, *a, dtype=dtype, **kw)
        used = sum(x() is not None and x().numel() * x().element_size() or 0 for x in live)
        if used + t.numel() * t.element_size() > room[0]:
            raise torch.OutOfMemoryError("no room")
        live.append(weakref.ref(t))
        return t

    live = []
    room[0] = 1 << 40
    monkeypatch.setattr(torch, "empty", small_device)
    plan = output_plan(2, workspace_limit=0)
    total = sum(x().numel() * x().element_size() for x in live if x() is not None)
    del plan
    live.clear()
    room[0] = total
    plan = output_plan(2)
    assert not plan.grouped and plan.workspace.numel() == one_shard_bytes(2)


@pytest.mark.parametrize("algorithm", [1, 2])
def test_output_plan_on_a_device_without_room_for_all_shards(monkeypatch, algorithm):
    # what one shard at a time had room for still runs
    limit, empty = one_shard_bytes(algorithm), torch.empty

    def full_device(shape, *a, dtype=None, **kw):
        if dtype == torch.uint8 and shape[0] > limit:
            raise torch.OutOfMemoryError("no room")
        return empty(shape, *a, dtype=dtype, **kw)

    monkeypatch.setattr(torch, "empty", full_device)
    plan = output_plan(algorithm)
    assert not plan.grouped and plan.workspace.numel() == limit


def test_a_single_shard_takes_the_single_calls(monkeypatch, embed_calls):
    fwd = []
    monkeypatch.setattr(B, "vp_embed_fwd", lambda *a: fwd.append("one"))
    monkeypatch.setattr(B, "vp_embed_fwd_group", lambda *a: fwd.append("group"))
    for p in (1, 2):
        plan = driver.EmbeddingPlan([torch.zeros(6, 8) for _ in range(p)], torch.zeros(5, dtype=torch.int64), torch.zeros(5, 8))
        plan.forward()
        plan.backward()
    assert fwd == ["one", "group"] and [c[0] for c in embed_calls] == ["one", "group"]

    def plan(N, h, rows, dtype, p=1, **kw):
        return driver.OutputLayerPlan(torch.zeros(N, h, dtype=dtype), [torch.zeros(rows, h, dtype=dtype) for _ in range(p)],
                                      torch.zeros(N, dtype=torch.int64), **kw)
    assert plan(512, 2048, 8000, torch.bfloat16).grouped              # dH in K slices: the group call alone has them
    assert not plan(512, 64, 256, torch.bfloat16).grouped             # no slices: nothing to gain
    assert not plan(128, 256, 4096, torch.float32).grouped            # fp32: the single call cuts K itself
    assert not plan(512, 64, 256, torch.bfloat16, 2, vocab_size=200).grouped      # the other shard is padding
    assert plan(512, 64, 256, torch.bfloat16, 2).grouped
