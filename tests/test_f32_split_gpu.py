"""fp32 launches of few rows: workgroups of 32 rows whose wavefronts (eight up to 64 columns, four above) stream
their sub-tiles of 32 rows by themselves, operands as three bf16 terms.  Against fp64 over the allowed pairs at the
edges of the sub-tiles, of a round of the wavefronts (4 and 8 sub-tiles) and of the columns (32, 64, 128 computed, chunks
of four), single steps on a running state, with grouped heads, infinities and NaN; the bounds are the fp32
configuration's."""
import pytest
import torch

from paper_2311_09431_amd import binding as sa
from tests import routes
from tests import test_nonfinite_gpu as nf

pytestmark = [pytest.mark.gpu, nf.np_quiet]

ROUTES = [
    # H, H_kv, c, d, dtype
    (1, 1, 17, 4, torch.float32),
    (2, 2, 32, 32, torch.float32),
    (2, 1, 33, 36, torch.float32),
    (1, 1, 129, 128, torch.float32),
    (3, 3, 160, 100, torch.float32),
    (2, 2, 257, 64, torch.float32),
    (4, 2, 289, 28, torch.float32),
]


def reached(route):
    H, Hkv, c, d, _ = route
    return all(routes._ask("f32x3_split_wanted", routes.args(c, d, H, Hkv), back) for back in (False, True))


@pytest.mark.parametrize("block", nf.BLOCKS)
@pytest.mark.parametrize("route", ROUTES)
def test_steps(route, block):
    assert reached(route)
    clean = lambda t, at: {"clean": lambda x: None}
    nf.check_forward_step(route, block, clean)
    nf.check_backward_step(route, block, clean)


@pytest.mark.parametrize("route", [ROUTES[2], ROUTES[3], ROUTES[5]])
def test_infinities_and_nan(route):
    for block in nf.BLOCKS:
        nf.check_forward_step(route, block, lambda t, at: {**nf.swallowed(t, at), **nf.masked(t, at)})
        nf.check_backward_step(route, block, nf.backward_kinds)


def test_rows_out_of_reach_are_others():
    # 32-bit byte offsets: the walk's last requests name up to 32 rows behind the last sub-tile
    for c, d in ((64, 64), (1000, 128)):
        behind = (c + 31) // 32 * 32 + 31
        for side in ("stride_s", "kv_stride_s"):
            pitches = [4 * ((1 << 31) // 16 // behind * i // 1000) for i in range(900, 1101)]
            taken = [p for p in pitches if routes._ask("f32x3_split_wanted", routes.args(c, d, 1, **{side: p}), False)]
            assert taken and all(behind * 4 * p + 4 * d + 4096 < 1 << 31 for p in taken)
            assert len(taken) < len(pitches)
