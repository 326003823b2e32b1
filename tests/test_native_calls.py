"""The binding's per-token calls (csrc/native.cpp): the checks and conversions of their arguments, without a GPU."""
import inspect

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


@pytest.mark.parametrize("args", [
    (0, "1"), (0.5, 1), (None, 1),
])
def test_whole_numbers(args):
    with pytest.raises(TypeError):
        rs.rat_scan(_shape(), *[None] * 7, *args)


def test_a_shape_is_a_shape():
    for s in (3, b"12", None):
        with pytest.raises(TypeError):
            rs.rat_scan(s, *[None] * 7, 0, 1)
