"""Backward above 128 columns with both column halves of dK and dV in one workgroup (full blocks of more than
128 key tiles, triangular ones and rings of more than 256): single steps against the oracle on both sides of
these rules and at the edges of its 32-row stages, with last tiles of a few rows, columns short of both
halves, grouped heads; and the ring drivers.  Coarse tile skipping, rows with gaps, interleaved heads and NaN on
this route are in test_tiled_gpu, test_strides_gpu and test_nonfinite_gpu."""
import pytest
import torch

from paper_2311_09431_amd import binding as sa
from tests import test_bwd_routes_gpu as routes
from tests import test_ring_walk_gpu as walks

pytestmark = pytest.mark.gpu

STEPS = [
    # B, H, H_kv, c, d                key tiles
    (1, 64, 64, 256, 256),          # 128: column halves side by side (full block)
    (1, 65, 65, 130, 136),          # 130, last tile of two rows (triangular: up to 256 halves side by side)
    (2, 35, 35, 161, 200),          # 140, one row into a stage
    (1, 32, 16, 1121, 144),         # 144, two heads per key/value head
    (1, 257, 257, 128, 256),        # 257: triangular blocks too
    (1, 104, 52, 545, 192),         # 260
]


@pytest.mark.parametrize("q_dev,kv_dev,layout", [(1, 0, sa.STRIPED), (0, 1, sa.STRIPED), (1, 0, sa.CONTIGUOUS)])
@pytest.mark.parametrize("B,H,Hkv,c,d", STEPS)
def test_steps_against_the_oracle(B, H, Hkv, c, d, q_dev, kv_dev, layout):
    routes.test_step_against_the_oracle(B, H, Hkv, c, d, q_dev, kv_dev, layout)


@pytest.mark.parametrize("layout", [sa.CONTIGUOUS, sa.STRIPED])
@pytest.mark.parametrize("H,Hkv,c,d,N", [(44, 44, 257, 152, 2), (88, 88, 128, 256, 3)])
def test_drivers_against_the_oracle(layout, H, Hkv, c, d, N):
    walks.test_drivers_against_the_oracle(layout, H, Hkv, c, d, N, torch.bfloat16)
