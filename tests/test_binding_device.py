"""Calls of the binding run on the device of their handle or tensors, whatever the current one is, and leave that as it was.  The
library and the devices are stand-ins: this is about what the binding does around them."""
import contextlib
import ctypes
import types

import numpy as np
import pytest
import torch

from paper_2311_02909_amd import bms


class FakeTensor:
    def __init__(self, shape, dtype, index):
        self.shape, self.dtype, self.device, self.is_cuda = shape, dtype, types.SimpleNamespace(index=index), True

    def dim(self):
        return len(self.shape)

    def is_contiguous(self):
        return True

    def data_ptr(self):
        return 4096


@pytest.fixture
def seen(monkeypatch):
    """Two devices, the current one 0; every library call as (device, current stream of it, stream given)."""
    now, calls = {"device": 0, "streams": {0: 100, 1: 101}}, []

    @contextlib.contextmanager
    def device(d):
        before, now["device"] = now["device"], getattr(d, "index", d)
        yield
        now["device"] = before

    @contextlib.contextmanager
    def stream(s):
        at = s.device
        before, now["streams"][at] = now["streams"][at], s.cuda_stream
        with device(at):
            yield
        now["streams"][at] = before

    def note(given):
        calls.append((now["device"], now["streams"][now["device"]], given))

    def current(d=None):
        at = now["device"] if d is None else getattr(d, "index", d)
        return types.SimpleNamespace(cuda_stream=now["streams"][at], device=at)

    def sizes(handle, h, view):
        view._obj.rows, view._obj.nnz, view._obj.ncols = 3, 5, 4
        return bms.OK

    def sample(*args):
        note(args[7])
        return bms.OK, 0    # (nothing to free)
    library = types.SimpleNamespace(bms_fetch_features=lambda *a: note(a[-1]) or bms.OK, bms_result_hop=sizes, bms_free=lambda h: None,
                                    bms_aggregate_hop=lambda *a: note(a[-1]) or bms.OK, bms_result_info=lambda *a: bms.OK)
    for name, value in (("current_device", lambda: now["device"]), ("device", device), ("stream", stream), ("current_stream", current),
                        ("ExternalStream", lambda s: types.SimpleNamespace(cuda_stream=s, device=now["device"])),
                        ("default_stream", lambda: types.SimpleNamespace(cuda_stream=0, device=now["device"]))):
        monkeypatch.setattr(torch.cuda, name, value)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda d: now["streams"][d], raising=False)
    monkeypatch.setattr(torch, "empty", lambda shape, dtype, device: note("empty") or FakeTensor(shape, dtype, device.index))
    monkeypatch.setattr(bms, "lib", lambda: library)
    monkeypatch.setattr(bms, "native", lambda: types.SimpleNamespace(sample=sample))
    yield now, calls
    assert now == {"device": 0, "streams": {0: 100, 1: 101}}   # as they were


@pytest.mark.parametrize("index", [0, 1])
@pytest.mark.parametrize("stream", [None, 555, 0])
def test_device_of_the_call(seen, index, stream):
    now, calls = seen
    csr = types.SimpleNamespace(device=index, handle=ctypes.c_void_p(8))
    wanted = 100 + index if stream is None else stream
    res = bms.sample_nodewise(csr, np.zeros((2, 3), dtype=np.int32), (4,), 1, stream=stream)
    bms.sample_ladies(csr, np.zeros((2, 3), dtype=np.int32), (4,), 1, stream=stream, recycle=res)
    assert res.device == index
    H, ids = FakeTensor((9, 16), torch.float32, index), FakeTensor((4,), torch.int32, index)
    bms.fetch_features(H, ids, stream=stream)
    bms.aggregate_hop(res, 0, FakeTensor((4, 16), torch.float32, index), stream=stream)
    assert {device for device, _, _ in calls} == {index}
    assert [given for _, _, given in calls if given != "empty"] == [wanted] * 4
    # allocations are made with the call's stream as the current one of its device
    assert [x[:2] for x in calls if x[2] == "empty"] == [(index, wanted)] * 2
