"""The native checks of the binding accept and refuse what the checks in Python do, and find the same addresses and stream."""
import ctypes

import pytest
import torch

pytestmark = pytest.mark.gpu


class Sub(torch.Tensor):
    pass


def test_native_checks_equal_the_python_checks(monkeypatch):
    import paper_2411_05288_amd.binding as B
    B.load_library()
    host = B._HOST
    assert host is not None
    f, bf = (torch.float32,), B._BF16_LIKE
    x = torch.zeros(6, 8, device="cuda")
    tensors = [x, x[2:], x[:, :4], x.t(), x[0], x[:0], x.bfloat16(), x.view(torch.int32), x.cpu(), torch.nn.Parameter(x),
               x.as_subclass(Sub), x.to_sparse(), x.half(), x[:1, :1], torch.zeros((), device="cuda"), None]
    native, python = 0, []
    for t in tensors:
        for dtypes in (None, f, bf):
            for shape in (None, (6, 8), torch.Size((6, 8)), (8, 6), (8,), (1, 1), ()):
                results = []
                for h in (host, None):
                    monkeypatch.setattr(B, "_HOST", h)
                    try:
                        results.append(B._ptr(t, "t", dtypes, shape))
                    except (B.VPError, RuntimeError) as e:
                        results.append(type(e))
                assert results[0] == results[1], (t, dtypes, shape)
                if t is not None and host.ptr(t, dtypes, shape) is not None:
                    native += 1
                python.append(results[1])
    assert native >= 30 and any(isinstance(r, type) for r in python)      # both answers occur
    ts = [x, x[:3], x[3:]]
    shapes = [tuple(t.shape) for t in ts]
    a = (ctypes.c_uint64 * 3).from_buffer_copy(host.ptrs(ts, f, shapes))
    assert list(a) == [t.data_ptr() for t in ts]
    assert host.ptrs(ts, f, (6, 8)) is None and host.ptrs(ts, f, shapes[:2]) is None
    assert host.same_shapes(ts[1:]) and not host.same_shapes(ts)
    monkeypatch.setattr(B, "_HOST", host)
    s = torch.cuda.Stream()
    assert B._stream(None) == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(s):
        assert B._stream(None) == s.cuda_stream
