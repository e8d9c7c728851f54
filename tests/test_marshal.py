"""Argument marshalling of the hot entry points (csrc/marshal.cpp): what it refuses, without a GPU."""
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
    for axis in (3, -4):
        with pytest.raises(IndexError):
            sa.sa_stripe_permute(x, x.clone(), 2, axis)


def test_counts_and_addresses():
    sa.lib()
    with pytest.raises(TypeError, match="arguments expected"):
        sa._marshal.two(0, 1)
    # as the library's own address
    assert sa._entry["sa_finalize"] == ctypes.cast(sa.lib().sa_finalize, ctypes.c_void_p).value
