"""Byte offsets of the tiles that the backward kernels with a ring of tiles request (csrc/sa_internal.h, TileByte, compiled for the
host): at the widest row strides that the 128-row kernels take, also the three requests behind the walk's end."""
import ctypes

import numpy as np
import pytest

from paper_2311_09431_amd import binding as sa
from tests import host_code
from tests import routes

MOST, ROWS = 1 << 31, 64
SOURCE = """
#include "sa_internal.h"
extern "C" void walk(int pitch, int tiles, int requests, int* at) {
    sa::TileByte byte{0, pitch};
    byte.block(0);
    for (int t = 0; t < requests; ++t) {        // as the kernels go on
        at[t] = byte.at;
        byte.next();
        if (t + 1 >= tiles) byte.stop();
    }
}
"""


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    return host_code.library(tmp_path_factory.mktemp("requests"), SOURCE).walk


@pytest.mark.parametrize("d", [68, 100, 128])
@pytest.mark.parametrize("c", [128, 129, 250, 1000, 8192])
def test_offsets_at_the_end_of_reach(walk, c, d):
    padded = (c + 127) // 128 * 128
    widest = max(pitch for pitch in range(MOST // 2 // padded // 8 * 8 - 256, MOST // 2 // padded // 8 * 8 + 257, 8)
                 if routes._ask("bwd_mfma_supported", routes.args(c, d, 1, kv_stride_s=pitch), sa.BF16))
    tile_pitch = ROWS * 2 * widest
    for tiles in ((c + ROWS - 1) // ROWS, padded // ROWS):          # of a walk over queries; over keys, in pairs
        at = np.zeros(tiles + 3, np.int32)
        walk(tile_pitch, tiles, tiles + 3, ctypes.c_void_p(at.ctypes.data))
        assert at[:tiles].tolist() == [t * tile_pitch for t in range(tiles)]
        assert all(tiles * tile_pitch == x < MOST for x in at[tiles:].tolist())
