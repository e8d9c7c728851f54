"""Byte offsets of the tiles that the backward kernels with a ring of tiles request (csrc/sa_internal.h, next_tile_byte, compiled
for the host): at the widest row strides that the 128-row kernels take, also the three requests behind the walk's end."""
import ctypes

import pytest

from paper_2311_09431_amd import binding as sa
from tests import host_code
from tests import routes

MOST, ROWS = 1 << 31, 64
SOURCE = """
#include "sa_internal.h"
extern "C" int next(int at, int pitch, int in_block) { return sa::next_tile_byte(at, pitch, in_block != 0); }
"""


@pytest.fixture(scope="module")
def next_tile(tmp_path_factory):
    return host_code.library(tmp_path_factory.mktemp("requests"), SOURCE).next


@pytest.mark.parametrize("d", [68, 100, 128])
@pytest.mark.parametrize("c", [128, 129, 250, 1000, 8192])
def test_offsets_at_the_end_of_reach(next_tile, c, d):
    padded = (c + 127) // 128 * 128
    widest = max(pitch for pitch in range(MOST // 2 // padded // 8 * 8 - 256, MOST // 2 // padded // 8 * 8 + 257, 8)
                 if routes._ask("bwd_mfma_supported", routes.args(c, d, 1, kv_stride_s=pitch), sa.BF16))
    tile_pitch = ROWS * 2 * widest
    for tiles in ((c + ROWS - 1) // ROWS, padded // ROWS):          # of a walk over queries; over keys, in pairs
        at, offsets = 0, []
        for t in range(tiles + 3):
            offsets.append(at)
            at = next_tile(ctypes.c_int(at), ctypes.c_int(tile_pitch), int(t + 1 < tiles))
        assert offsets[:tiles] == [t * tile_pitch for t in range(tiles)]
        assert all(0 <= x < MOST for x in offsets) and offsets[tiles:] == [0, 0, 0]
