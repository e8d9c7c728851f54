"""Argument marshalling of the hot entry points (csrc/marshal.cpp): what it refuses, and the axes of a permutation."""
import ctypes

import pytest
import torch

from paper_2311_09431_amd import binding as sa


def tensors(n):
    return [torch.zeros(1, 1, 8, 4) for _ in range(n)]


def shape():
    return sa.shard_shape(torch.zeros(1, 1, 8, 4), 8)


def calls(shape, t=tensors):
    return [
        lambda: sa.sa_state_init(*t(2), shape),
        lambda: sa.sa_finalize(*t(2), shape),
        lambda: sa.sa_bwd_preprocess(*t(3), shape),
        lambda: sa.sa_attn_step_fwd(*t(5), 0, 0, 1, sa.STRIPED, shape),
        lambda: sa.sa_attn_step_bwd(*t(9), 0, 0, 1, sa.STRIPED, shape),
        lambda: sa.sa_ring_fwd(*t(5), 1, sa.STRIPED, shape),
        lambda: sa.sa_ring_bwd(*t(10), 1, sa.STRIPED, shape),
        lambda: sa.sa_rope(*t(2), torch.zeros(8, dtype=torch.int32), shape),
        lambda: sa.sa_stripe_permute(*t(2), 2),
    ]


def test_tensors_off_the_gpu_and_other_objects():
    sa.lib()
    for call in calls(shape()):
        with pytest.raises(TypeError, match="GPU tensor"):
            call()
    for call in calls(shape(), lambda n: [None] * n)[:7]:
        with pytest.raises(TypeError, match="GPU tensor"):
            call()


def test_permute_looks_at_its_tensors_first():
    x = torch.zeros(2, 8, 4)
    for other in (x.transpose(0, 2), torch.zeros(2, 8, 2), x.to(torch.int32)):
        with pytest.raises(ValueError):
            sa.sa_stripe_permute(x, other, 2, 1)
        with pytest.raises(ValueError):
            sa.sa_unstripe_permute(other, x, 2, 1)
    for axis in (3, -4, 1 << 64, -(1 << 64)):
        with pytest.raises(IndexError):
            sa.sa_stripe_permute(x, x.clone(), 2, axis)
    with pytest.raises(TypeError):
        sa.sa_stripe_permute(x, x.clone(), 2, 1.0)


@pytest.mark.parametrize("shape", [(8,), (6, 4), (2, 8, 4), (3, 1, 5, 2)])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_a_permutation_stays_inside_its_tensor(shape, dtype):
    # from whichever end the axis is counted: what is moved is the tensor, the rows along that axis
    sa.lib()
    x = torch.zeros(shape, dtype=dtype)
    for axis in range(-len(shape), len(shape)):
        outer, rows, inner = sa._marshal.extent_of(x, axis)
        assert rows == shape[axis] and outer * rows * inner == x.numel() * x.element_size()
        assert inner == x.stride(axis) * x.element_size()


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32, torch.int32])
def test_axes_counted_from_the_end(dtype):
    x = torch.arange(2 * 6 * 12, device="cuda").view(2, 6, 12).to(dtype)
    for axis in (-1, -2):
        y, want, back = (torch.empty_like(x) for _ in range(3))
        sa.sa_stripe_permute(x, y, 3, axis)
        sa.sa_stripe_permute(x, want, 3, axis + 3)
        sa.sa_unstripe_permute(y, back, 3, axis)
        assert torch.equal(y, want) and torch.equal(back, x)
        assert not torch.equal(y, x)


def test_counts_and_addresses():
    sa.lib()
    with pytest.raises(TypeError, match="arguments expected"):
        sa._marshal.two(0, 1)
    # as the library's own address
    assert sa._entry["sa_finalize"] == ctypes.cast(sa.lib().sa_finalize, ctypes.c_void_p).value


def test_a_binding_without_its_extension_says_how_to_build(monkeypatch):
    # not there, or for another torch: each entry point, and the library's first use
    s = shape()
    monkeypatch.setattr(sa, "_marshal", sa._NotBuilt("no module"))
    for call in calls(s):
        with pytest.raises(RuntimeError, match="paper_2311_09431_amd.build.*no module"):
            call()
    monkeypatch.setattr(sa, "_lib", None)
    with pytest.raises(RuntimeError, match="paper_2311_09431_amd.build.*no module"):
        sa.lib()


class AsParameter:
    def __init__(self, x):
        self._as_parameter_ = x


class Index:
    def __index__(self):
        return 2


TWO = [2, True + 1, Index(), ctypes.c_int32(2), AsParameter(Index()), AsParameter(ctypes.c_int32(2))]


def test_integers_are_what_ctypes_takes_for_them():
    x = torch.zeros(2, 8, 4)
    f = ctypes.CFUNCTYPE(ctypes.c_int, ctypes.c_int32)(lambda n: n)
    for n in TWO:
        assert f(n) == 2
        with pytest.raises(TypeError, match="GPU tensor"):      # the number has been taken
            sa.sa_stripe_permute(x, x.clone(), n, 1)
    for n in (2.0, "2", None, ctypes.c_int64(2), AsParameter(2.0)):
        with pytest.raises(ctypes.ArgumentError):
            f(n)
        with pytest.raises(ctypes.ArgumentError):
            sa.sa_stripe_permute(x, x.clone(), n, 1)


@pytest.mark.gpu
def test_a_step_with_such_integers():
    q, k, v = (torch.randn(1, 1, 8, 4, device="cuda") for _ in range(3))
    got = []
    for two in TWO:
        o, lse = torch.zeros_like(q), torch.full((1, 1, 8), -float("inf"), device="cuda")
        s = sa.shard_shape(q, 8, lse)
        sa.sa_attn_step_fwd(q, k, v, o, lse, two, 1, 3, ctypes.c_int32(sa.STRIPED), s)
        got.append(torch.cat((o.flatten(), lse.flatten())))
    assert all(torch.equal(g, got[0]) for g in got)
