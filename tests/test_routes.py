"""Host-side rules of the dispatch: which calls the kernels that address rows through 32-bit byte offsets
take (no GPU needed)."""
import pytest

from paper_2311_09431_amd import binding as sa
from tests import routes

MOST = 1 << 31          # byte offsets below it


def test_ordinary_calls():
    # (what the strides below are measured against; also that the mirrored struct is the library's)
    assert routes.forward(routes.args(128, 128, 1)) == "split"
    assert routes.forward(routes.args(4096, 128, 32)) == "128 rows"
    assert routes.forward(routes.args(127, 128, 1)) == "short"
    assert routes.forward(routes.args(128, 132, 1)) == "fp32"
    assert routes.forward(routes.args(128, 128, 1), sa.F32) == "fp32"
    assert routes.backward(routes.args(128, 128, 1)) == "split"
    assert routes.backward(routes.args(4096, 128, 32)) == "128 rows"
    assert routes.backward(routes.args(127, 128, 1)) == "short"
    assert routes.forward(routes.args(1024, 128, 2, N=4, layout=sa.CONTIGUOUS)) == "split"


@pytest.mark.parametrize("d", [64, 100, 128])
@pytest.mark.parametrize("c", [128, 160, 8192])
def test_wide_query_rows_stay_with_the_kernel_that_reads_them_by_pointer(c, d):
    # 128-row workgroups read Q by 64-bit pointers and take any row stride; the split ones go through a descriptor
    for pitch in (MOST // 2 // c + 8, MOST // c + 8, MOST // 2 + 8):
        assert routes.forward(routes.args(c, d, 1, stride_s=pitch)) == "128 rows"
        assert routes.backward(routes.args(c, d, 1, stride_s=pitch)) == "fp32"
    # and keys as far apart: neither
    assert routes.forward(routes.args(c, d, 1, kv_stride_s=MOST // 2 // c + 8)) == "fp32"


@pytest.mark.parametrize("c", [1, 33, 97, 127, 128, 129, 160, 8192])
@pytest.mark.parametrize("side", ["stride_s", "kv_stride_s"])
def test_every_offset_of_a_split_launch_is_below_the_limit(c, side):
    # the split kernels' last requests name the 32 rows behind the block's last sub-tile, 16 and 16
    d, behind = 64, (c + 31) // 32 * 32 + 31
    taken = []
    for pitch in range(8 * (MOST // 2 // (c + 160) // 8) - 64, 8 * (MOST // 2 // c // 8) + 65, max(8, 8 * (MOST // 2 // c // 8 // 4096))):
        for ask in (routes.forward, routes.backward):
            if ask(routes.args(c, d, 1, **{side: pitch})) in ("split", "short"):
                taken.append(pitch)
                assert behind * 2 * pitch + 2 * d < MOST, (ask.__name__, pitch)
    assert taken or c == 1          # the rule is not empty there


def test_split_rules_at_their_edges():
    # where the measured lines lie (the figures stand at the rules)
    bwd = lambda H, c, d, layout=sa.STRIPED, **kw: routes.backward(routes.args(c, d, H, layout=layout, **kw))     # noqa: E731
    assert bwd(32, 512, 64, sa.CONTIGUOUS) == "split" and bwd(32, 512, 32, sa.CONTIGUOUS) == "128 rows"
    assert bwd(20, 512, 32, sa.CONTIGUOUS) == "split"
    assert bwd(32, 2048, 64) == "128 rows" and bwd(31, 2048, 64) == "split" and bwd(32, 1024, 64) == "split"
    assert bwd(32, 1024, 64, sa.CONTIGUOUS, N=2) == "128 rows"
    # key/value heads, a nearly empty last tile counting for them
    assert bwd(40, 128, 96, sa.CONTIGUOUS) == "split" and bwd(41, 128, 96, sa.CONTIGUOUS) == "128 rows" and bwd(64, 128, 96) == "split"
    assert bwd(64, 768, 128, Hkv=16) == "split" and bwd(68, 768, 128, Hkv=17) == "128 rows" and bwd(68, 672, 128, Hkv=17) == "split"
    assert bwd(96, 512, 128, sa.CONTIGUOUS, Hkv=24) == "split" and bwd(100, 512, 128, sa.CONTIGUOUS, Hkv=25) == "128 rows"
    assert bwd(224, 512, 64, Hkv=56) == "split" and bwd(228, 512, 64, Hkv=57) == "128 rows" and bwd(228, 416, 64, Hkv=57) == "split"
    fwd = lambda H, c, d, Hkv=None: routes.forward(routes.args(c, d, H, Hkv, layout=sa.CONTIGUOUS))               # noqa: E731
    assert fwd(15, 1024, 128) == "128 rows" and fwd(15, 1024, 64) == "split" and fwd(14, 1152, 128) == "split"
    assert fwd(9, 1700, 128) == "split" and fwd(15, 1024, 128, 3) == "split"
    # short blocks of many heads, few columns: one forward block, not the backward or a walk over several
    for H, c, d, route in ((512, 32, 32, "short"), (513, 32, 32, "fp32"), (384, 33, 32, "short"), (385, 33, 32, "fp32"), (1000, 33, 36, "short")):
        assert fwd(H, c, d) == route and bwd(H, c, d) == "short"
        assert routes.forward(routes.args(c, d, H, N=2)) == "short"


@pytest.mark.parametrize("H,Hkv,c,N,route", [
    (8, 8, 1024, 4, "split"), (4, 4, 4096, 4, "split"), (32, 8, 1024, 8, "split"), (16, 16, 2048, 2, "split"),
    (32, 32, 512, 2, "128 rows"), (33, 33, 1024, 2, "128 rows")])
def test_narrow_backward_of_one_device_against_all_shards(H, Hkv, c, N, route):
    # the queries of one device fill the chip's 256 compute units with 128-row tiles only where they are as many as that
    a = routes.args(c, 32, H, Hkv, N=N)
    a.n_q, a.q_dev = 1, N - 1
    assert routes.backward(a) == route


@pytest.mark.parametrize("H,Hkv,c,N,d,ranks", [
    (32, 32, 1024, 4, 128, False), (64, 64, 1024, 4, 100, False), (32, 32, 512, 8, 256, False), (32, 32, 2048, 2, 256, False),
    (24, 24, 512, 8, 256, False), (16, 16, 4096, 4, 128, True), (32, 32, 4096, 2, 64, True), (24, 24, 1000, 4, 100, True),
    (64, 64, 1024, 2, 64, True), (64, 64, 1024, 2, 128, False), (32, 32, 1024, 8, 32, True), (32, 32, 1024, 8, 64, False),
    (32, 8, 4096, 4, 128, True)])
def test_keys_of_one_device_against_all_shards_by_ranks_only_where_walks_are_long(H, Hkv, c, N, d, ranks):
    a = routes.args(c, d, H, Hkv, N=N)
    whole = a.H_kv * N * ((c + 127) // 128)
    assert routes.keys_by_rank(a) == (512 < whole <= (1535 if d > 128 else 2560))
    a.n_q, a.q_dev = 1, N - 1
    assert routes.keys_by_rank(a) == ranks


def test_wide_walks_over_a_striped_ring_go_by_ranks_up_to_six_rounds():
    ranks = lambda c, d, H, **kw: routes.queries_by_rank(routes.args(c, d, H, **kw))     # noqa: E731
    assert ranks(1024, 256, 48, N=4) and not ranks(1024, 256, 49, N=4) and not ranks(1000, 136, 64, N=4)
    assert ranks(1024, 256, 64, N=4, layout=sa.CONTIGUOUS) and ranks(4096, 256, 64) and not ranks(4096, 256, 65)
    assert ranks(1024, 128, 80, N=4) and not ranks(1024, 128, 81, N=4) and ranks(1024, 112, 96, N=4)


@pytest.mark.parametrize("d,few,most", [(64, 3, 256), (100, 3, 192), (128, 3, 192), (256, 3, 512), (32, 1, 768), (28, 3, 256)])
def test_many_heads_of_few_tiles_stay_in_groups(d, few, most):
    ranks = lambda tiles, H: routes.queries_by_rank(routes.args(128 * tiles, d, H))     # noqa: E731
    assert ranks(few + 1, min(160, most) if few > 1 else 600)
    assert few == 1 or not ranks(few, 192)
    tiles = 4 if few > 1 else 2
    assert ranks(tiles, most) and not ranks(tiles, most + 1)


def test_wide_keys_go_by_ranks_further_where_heads_have_few_tiles():
    ranks = lambda tiles, H: routes.keys_by_rank(routes.args(128 * tiles, 256, H))     # noqa: E731
    assert ranks(4, 512) and not ranks(4, 513) and ranks(8, 192) and not ranks(8, 193) and ranks(9, 170) and not ranks(16, 96)


@pytest.mark.parametrize("H,c,route", [
    (32, 1024, "128 rows"), (16, 2048, "128 rows"), (8, 4096, "split"), (8, 3000, "split"), (12, 3000, "split"),
    (16, 3000, "split"), (20, 3000, "128 rows"), (64, 512, "128 rows"), (24, 1024, "128 rows"), (5, 8192, "split")])
def test_narrow_backward_of_one_step(H, c, route):
    assert routes.backward(routes.args(c, 32, H)) == route


@pytest.mark.parametrize("backward", [False, True])
def test_a_split_fp32_launch_holds_fewer_threads_than_hip_takes(backward):
    # workgroups of 32 rows, 512 threads up to 64 columns and 256 above; the rule takes the longest walks of the most heads
    # up to 32 columns
    taken = []
    for d, threads in ((4, 512), (32, 512), (64, 512), (128, 256)):
        for H, Hkv, N, layout in ((65535, 65535, 1, sa.STRIPED), (65535, 65535, 1, sa.CONTIGUOUS), (65535, 4369, 1, sa.STRIPED),
                                  (8192, 8192, 8, sa.STRIPED), (32767, 1, 1, sa.STRIPED), (1024, 1, 16, sa.CONTIGUOUS)):
            for c in (17, 40, 100, 129, 1000, 2048, 2080, 2112, 4096, 1 << 14, 1 << 17, 1 << 20):
                a = routes.args(c, d, H, Hkv, layout=layout, N=N)
                if routes.f32(a, backward) == "split":
                    workgroups = (c + 31) // 32 * N * (H + (Hkv if backward else 0))
                    assert workgroups * threads < 1 << 32, (d, H, Hkv, N, c)
                    taken.append(workgroups * threads)
    assert max(taken) > 1 << 30         # (it is not that large launches are never taken)


def test_backward_in_one_launch_at_its_edges():
    one = lambda H, c, d=128, Hkv=None, **kw: routes.one_launch(routes.args(c, d, H, Hkv, **kw))     # noqa: E731
    full = dict(layout=sa.CONTIGUOUS)
    # key tiles of uneven work; up to 64 columns and above 128 (two workgroups a tile) as many as compute units
    assert one(12, 4096) and one(32, 1500) and not one(35, 1400) and one(384, 128) and not one(385, 128, 68)
    assert one(160, 1024, 100, 40) and not one(164, 1024, 100, 41) and one(120, 1000, 112, 40)
    assert one(256, 128, 64) and not one(257, 128, 64) and one(256, 128, 256) and not one(257, 128, 136)
    # walks of more than five blocks, each of two or three tiles: up to a key tile per compute unit
    for c, short in ((128, False), (129, True), (256, True), (384, True), (385, False)):
        tiles = (c + 127) // 128
        kv = 257 // tiles + 1
        assert one(5 * kv, c, 96, kv) and one(6 * kv, c, 96, kv) != short and one(8 * (256 // tiles), c, 96, 256 // tiles)
        assert one(3 * (kv // 2 + 1), c, 96, kv // 2 + 1, N=2) != short
    # workgroups of both kinds of a full block
    assert one(11, 2048, **full) and not one(12, 2048, **full) and one(176, 128, **full) and not one(177, 128, **full)
    assert one(128, 128, 64, **full) and not one(129, 128, 64, **full)


@pytest.mark.parametrize("layout", [sa.STRIPED, sa.CONTIGUOUS])
def test_backward_of_one_device_in_one_launch_at_its_edges(layout):
    def one(H, c, N, d=128):
        a = routes.args(c, d, H, N=N, layout=layout)
        a.n_q, a.q_dev = 1, N - 1
        return routes.one_launch(a)
    # one round of query tiles, eight of key tiles
    assert one(32, 1024, 8) and not one(33, 1024, 8) and one(128, 256, 8, 100) and not one(128, 256, 9, 100)
    assert not one(64, 1024, 4) and one(256, 128, 2, 68) and not one(257, 128, 2, 68)
