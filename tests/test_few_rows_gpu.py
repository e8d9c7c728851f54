"""Steps on blocks of up to 16 rows: a group of 16, 32 or 64 lanes owns a row.  Against fp64 over the allowed
pairs, at the sizes of the groups (64, 128, 256 columns), on both sides of the rule (8 rows, 16 for fp32
storage and above 128 columns; a group of heads counts in the backward), and with infinities and NaN."""
import pytest
import torch

from tests import test_nonfinite_gpu as nf

pytestmark = [pytest.mark.gpu, nf.np_quiet]

ROUTES = [
    # H, H_kv, c, d, dtype
    (1, 1, 3, 4, torch.float32),
    (5, 5, 8, 64, torch.bfloat16),
    (4, 2, 8, 68, torch.bfloat16),      # 16 queries a key
    (6, 2, 8, 36, torch.bfloat16),      # 24: the backward by the larger blocks' kernels
    (3, 3, 9, 64, torch.bfloat16),      # beyond the rule
    (3, 3, 16, 128, torch.float32),
    (3, 1, 5, 132, torch.float32),
    (2, 2, 16, 256, torch.bfloat16),
    (2, 2, 17, 256, torch.bfloat16),    # beyond the rule
]


@pytest.mark.parametrize("block", nf.BLOCKS)
@pytest.mark.parametrize("route", ROUTES)
def test_steps(route, block):
    clean = lambda t, at: {"clean": lambda x: None}
    nf.check_forward_step(route, block, clean)
    nf.check_backward_step(route, block, clean)


@pytest.mark.parametrize("block", nf.BLOCKS)
@pytest.mark.parametrize("route", ROUTES)
def test_infinities_and_nan(route, block):
    nf.check_forward_step(route, block, lambda t, at: {**nf.swallowed(t, at), **nf.masked(t, at)})
    nf.check_backward_step(route, block, nf.backward_kinds)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_one_row(dtype):
    for block in nf.BLOCKS:
        for d in (4, 64, 100, 256):
            nf.check_forward_step((2, 1, 1, d, dtype), block, lambda t, at: {"clean": lambda x: None})
            nf.check_backward_step((2, 1, 1, d, dtype), block, lambda t, at: {"clean": lambda x: None})
