"""The binding's per-token calls (csrc/native.cpp): the checks and conversions of their arguments, without a GPU."""
import ctypes
import inspect

import numpy as np
import pytest
import torch

from paper_2605_28640_amd import binding as rs


def _shape():
    return rs.make_shape(1, 2, 2, 64, 64, 16, torch.float32)


@pytest.mark.parametrize("name,names", [
    ("rat_scan", "s k v g state_k state_v k_cache v_cache t0 T_new ws meta"),
    ("sparse_attn_decode", "s q k_cache v_cache T_valid scale idx K meta n_first n_local out lse_out idx_out ws"),
    ("rat_decode_step", "s k v g state_k state_v k_cache v_cache meta q scale K n_first n_local T_max out lse_out idx_out ws"),
])
def test_signatures(name, names):
    assert list(inspect.signature(getattr(rs, name)).parameters) == names.split()


@pytest.mark.parametrize("bad", [torch.zeros(4), torch.zeros(4, 4).t(), torch.nn.Parameter(torch.zeros(2))])
def test_only_contiguous_device_tensors(bad):
    with pytest.raises(AssertionError):
        rs.rat_scan(_shape(), bad, *[None] * 6, t0=0, T_new=1)


class _Odd(torch.Tensor):
    @property
    def is_cuda(self):
        raise ValueError("asked")


def test_a_subclass_is_asked_the_way_it_always_was():
    with pytest.raises(ValueError, match="asked"):
        rs.rat_scan(_shape(), torch.zeros(4).as_subclass(_Odd), *[None] * 6, t0=0, T_new=1)


def _step(**change):
    """rat_decode_step with every argument of its plain type but those of `change`."""
    args = dict.fromkeys("k v g state_k state_v k_cache v_cache meta q out lse_out idx_out".split())
    args.update(s=_shape(), scale=0.125, K=1, n_first=0, n_local=0, T_max=16, ws=rs.Workspace.__new__(rs.Workspace))
    args["ws"].buf = torch.zeros(rs.RS_WS_CTRL_BYTES, dtype=torch.uint8)
    args.update(change)
    rs.rat_decode_step(**args)


# What ctypes refuses is refused with the exception that the library's other functions raise for it.  (The stream is looked up
# before ctypes looks at the arguments, and there is none without a GPU.)
@pytest.mark.parametrize("bad", ["1", 0.5, None, np.float32(1)])
@pytest.mark.parametrize("call", [
    lambda x: rs.rat_scan(_shape(), *[None] * 7, x, 1),
    lambda x: rs.rat_scan(_shape(), *[None] * 7, 0, x),
    lambda x: rs.quest_page_meta(_shape(), None, None, 0, x),
    lambda x: _step(K=x),
    lambda x: _step(T_max=x),
])
def test_whole_numbers(call, bad, monkeypatch):
    monkeypatch.setattr(rs, "_stream", lambda: 0)
    with pytest.raises(ctypes.ArgumentError):
        call(bad)


def _addresses():
    return [ctypes.cast(getattr(rs.load(), n), ctypes.c_void_p).value for n in ("rat_scan", "sparse_attn_decode", "rat_decode_step")]


def test_good_arguments_reach_the_library(monkeypatch):
    monkeypatch.setattr(rs, "_stream", lambda: 0)
    native = rs._calls()
    native.setup(*_addresses(), rs._check, lambda dev: 0, lambda: 0, rs.rs_shape, rs.Workspace)
    try:
        for call in (_step, lambda: _step(scale=1), lambda: _step(K=True), lambda: _step(K=np.int64(1)),
                     lambda: _step(T_max=torch.tensor(16)), lambda: rs.rat_scan(_shape(), *[None] * 7, 0, 1)):
            with pytest.raises(rs.RatsparseError):  # null caches: the library's own answer, before any launch
                call()
    finally:
        native.setup(*_addresses(), rs._check, torch._C._cuda_getCurrentRawStream, torch.cuda.current_device, rs.rs_shape, rs.Workspace)


class _Other(ctypes.Structure):
    _fields_ = rs.rs_shape._fields_


def test_a_shape_is_a_shape(monkeypatch):
    for s in (3, b"12", None, bytes(_shape()), np.zeros(7, np.int32)):
        with pytest.raises(TypeError):
            rs.rat_scan(s, *[None] * 7, 0, 1)
    monkeypatch.setattr(rs, "_stream", lambda: 0)
    with pytest.raises(ctypes.ArgumentError):
        rs.rat_scan(_Other(*[1] * 7), *[None] * 7, 0, 1)


def test_the_decode_calls_need_a_workspace():
    for ws in (None, 0):
        with pytest.raises(AttributeError):
            _step(ws=ws)
        with pytest.raises(AttributeError):
            rs.sparse_attn_decode(_shape(), None, None, None, 16, 0.125, None, 1, None, 0, 0, None, None, None, ws)
