"""Order of a backward launch that holds both kinds of workgroups, one to a compute unit (csrc/sa_internal.h, placed_kinds and
owns_keys, compiled for the host): every workgroup once, each kind heaviest first, the rarer kind on all 32 places alike, or (up to 64
columns and above 128, where it is not in step with them) evenly among the others."""
import ctypes

import numpy as np
import pytest

from paper_2311_09431_amd import binding as sa
from tests import host_code
from tests import routes

SOURCE = """
#include "sa_internal.h"
extern "C" void order(const sa::StepArgs* a, int keys, int queries, double ratio, int* owns, int* at, int* first) {
    const sa::PlacedKinds k = sa::placed_kinds(*a, keys, queries, ratio);
    first[0] = k.queries_first; first[1] = k.keys_first;
    for (int i = 0; i < keys + queries; ++i) { at[i] = i; owns[i] = sa::owns_keys(k, at[i]); }
}
"""


@pytest.fixture(scope="module")
def order(tmp_path_factory):
    fn = host_code.library(tmp_path_factory.mktemp("order"), SOURCE).order
    fn.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_int, ctypes.c_double] + [ctypes.c_void_p] * 3
    fn.restype = None

    def call(a, keys, queries, ratio):
        owns, at_, first = np.zeros(keys + queries, np.int32), np.zeros(keys + queries, np.int32), np.zeros(2, np.int32)
        fn(ctypes.byref(a), keys, queries, ratio, owns.ctypes.data, at_.ctypes.data, first.ctypes.data)
        return owns.astype(bool), at_, first
    return call


# tiles, heads, key/value heads, shards of keys (1: one step, the triangular block or the full one)
CASES = ([(t, kv * g, kv, 1, layout) for g in (1, 2, 3, 5, 7, 8, 15) for t, kv in ((1, 257), (3, 98), (8, 44), (5, 64), (1, 1))
          for layout in (sa.STRIPED, sa.CONTIGUOUS)]
         + [(t, kv * g, kv, n, layout) for n, g in ((6, 2), (12, 4), (14, 1), (14, 2), (3, 3), (16, 8)) for t, kv in ((1, 50), (4, 25), (15, 7))
            for layout in (sa.STRIPED, sa.CONTIGUOUS)])


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("tiles,H,Hkv,N,layout", CASES)
def test_order(order, tiles, H, Hkv, N, layout, d):
    a = routes.args(128 * tiles, d, H, Hkv, N=N, layout=layout)
    a.n_q, a.q_dev = 1, (N - 1 if N > 1 else a.q_dev)
    keys, queries = tiles * N * Hkv, tiles * H
    for ratio in (0., 1.45):
        owns, at, first = order(a, keys, queries, ratio)
        for mine, count in ((at[owns], keys), (at[~owns], queries)):        # all of them, heaviest first
            assert np.array_equal(mine, np.arange(count))
        front = int(first.sum())
        unit = 8 if (keys - first[1]) % 8 == 0 and (queries - first[0]) % 8 == 0 else 1
        rest = owns[front:front + (len(owns) - front) // unit * unit]
        rarer = rest if 2 * rest.sum() <= len(rest) else ~rest
        few, every = int(rarer.sum()) // unit, len(rarer) // unit
        if d == 128 or (few and every % few == 0 and every // few % 2 == 0):
            on = [int(rarer[place::32].sum()) for place in range(min(32, len(rarer)))]
            assert not on or max(on) - min(on) <= 1, on
        else:           # evenly
            where = np.flatnonzero(rarer[::unit])
            assert len(where) < 2 or np.ptp(np.diff(where)) <= 1
        # walks of queries that outlast all of keys lead (products: 3 to 4 a pair)
        assert first[0] == (queries if d == 128 and N > 1 and 3 * N >= 4 * (H // Hkv) else 0)


@pytest.mark.parametrize("group", [20000, 30000])
def test_a_large_group_evenly(order, group):
    # fewer than 2^24 workgroups, of 384 and 500 key/value heads; d 64
    heads = 384 if group == 30000 else 500
    a = routes.args(128, 64, heads * group, heads)
    owns, at, _ = order(a, heads, heads * group + 1, 0.)
    assert np.array_equal(at[owns], np.arange(heads)) and np.array_equal(at[~owns], np.arange(heads * group + 1))


def test_a_large_group(order):
    # 384 key-owning workgroups of 30000 query heads each: products of both pass 32 bits
    a = routes.args(128, 128, 384 * 30000, 384)
    owns, at, _ = order(a, 384, 384 * 30000, 0.)
    assert np.array_equal(at[owns], np.arange(384)) and np.array_equal(at[~owns], np.arange(384 * 30000))
    # in units of 8; the rate, 48 units in 360012 rows, is 2236 of 2^24 units a row, rounded down
    assert abs(np.diff(np.flatnonzero(owns)[::8]) - 8 * 30001).max() <= 64 + 8 * 30001 / 2236
