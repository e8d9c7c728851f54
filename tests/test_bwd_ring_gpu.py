"""The backward kernels with a ring of tiles (65 to 128 columns): walks of one tile and of few, last tiles of one row, partial
16-byte chunks, groups of heads, several shards in one walk, both kinds in one launch and each in its own, rows at the end of reach."""
import numpy as np
import pytest
import torch

from paper_2311_09431_amd import binding as sa
from paper_2311_09431_amd import inputs
from tests import helpers as hp
from tests import routes
from tests.test_bwd_routes_gpu import test_step_against_the_oracle as step_against_the_oracle

pytestmark = pytest.mark.gpu

STEPS = [
    # B, H, H_kv, c, d, one launch of both kinds for uneven work, for a full block, keys by ranks (uneven work)
    (1, 140, 140, 128, 128, True, True, False),         # walks of two tiles
    (1, 70, 70, 129, 100, True, True, False),           # a last tile of one row: a walk of one tile
    (2, 13, 13, 321, 68, True, True, False),            # 78 tiles, 65 rows behind the last whole one
    (1, 160, 40, 200, 112, True, False, False),         # four query heads in a walk
    (1, 231, 33, 1100, 100, True, False, False),        # 297 tiles, seven query heads: every eighth workgroup owns keys
    (1, 111, 37, 900, 124, True, False, False),         # 296 tiles, three query heads, in units of 8
    (1, 918, 153, 200, 80, False, False, False),        # 306 tiles, walks of six blocks of two
    (1, 130, 130, 257, 124, False, False, False),
    (1, 800, 400, 128, 72, False, False, False),        # two query heads in a walk
    (1, 130, 130, 513, 116, False, False, True),        # 650 tiles
]


@pytest.mark.parametrize("q_dev,kv_dev,layout", [(1, 0, sa.STRIPED), (0, 1, sa.STRIPED), (1, 0, sa.CONTIGUOUS), (1, 1, sa.CONTIGUOUS)])
@pytest.mark.parametrize("B,H,Hkv,c,d,uneven,full,ranks", STEPS)
def test_steps(B, H, Hkv, c, d, uneven, full, ranks, q_dev, kv_dev, layout):
    a = routes.args(c, d, H, Hkv, B, q_dev=q_dev, kv_dev=kv_dev, layout=layout)
    is_full = layout == sa.CONTIGUOUS and q_dev != kv_dev
    assert routes.backward(a) == "128 rows" and routes.one_launch(a) == (full if is_full else uneven)
    assert routes.keys_by_rank(a) == (ranks and not is_full)
    step_against_the_oracle(B, H, Hkv, c, d, q_dev, kv_dev, layout)


@pytest.mark.parametrize("layout", [sa.STRIPED, sa.CONTIGUOUS])
@pytest.mark.parametrize("H,Hkv,N,c,d,dev,one", [
    (24, 24, 3, 200, 96, -1, True), (24, 24, 3, 200, 96, 1, True), (70, 70, 3, 192, 128, -1, False), (18, 18, 4, 129, 100, 3, True),
    # grouped heads: a walk goes through the shards of a head, then to the next head
    (48, 24, 3, 200, 96, -1, True), (140, 70, 3, 192, 128, -1, False), (90, 30, 4, 129, 68, 2, True),
    # one device's queries against more key tiles than launches of both kinds hold otherwise: 1120 (striped) and 560
    (70, 70, 8, 129, 100, 7, True), (70, 70, 4, 192, 128, 3, True),
    # ... and more query tiles than compute units
    (130, 130, 4, 200, 120, 3, False)])
def test_walks_over_several_shards(H, Hkv, N, c, d, dev, one, layout):
    S, group = N * c, H // Hkv
    a = routes.args(c, d, H, Hkv, N=N, layout=layout)
    if dev >= 0:
        a.n_q, a.q_dev, a.n_kv = 1, dev, N if layout == sa.STRIPED else dev + 1
    assert routes.backward(a) == "128 rows" and routes.one_launch(a) == one
    q, k, v, g = (inputs.gaussian((1, h, S, d), 40 + d + i, torch.bfloat16) for i, h in enumerate((H, Hkv, Hkv, H)))
    x = [hp.to_device_order(t.cuda(), N, layout) for t in (q, k, v, g)]
    o, lse = torch.empty(1, H, S, d, device="cuda"), torch.empty(1, H, S, device="cuda")
    shape = sa.shard_shape(x[0], c, lse, kv=x[1] if Hkv != H else None)
    sa.sa_ring_fwd(*x[:3], o, lse, N, layout, shape)
    delta, grads = torch.empty_like(lse), [torch.full((1, h, S, d), float("nan"), device="cuda") for h in (H, Hkv, Hkv)]
    own = slice(dev * c, (dev + 1) * c) if dev >= 0 else slice(0, S)
    sa.sa_ring_bwd(*x, o, lse, delta, *grads, N, layout, shape, dev)
    torch.cuda.synchronize()
    # one device's part: dO of its own rows alone
    only = torch.zeros_like(x[3])
    only[:, :, own] = x[3][:, :, own]
    only = torch.from_numpy(hp.from_device_order_host(only.float().cpu().numpy(), N, layout)).to(torch.bfloat16)
    dq, dk, dv = (torch.from_numpy(hp.from_device_order_host(t.cpu().numpy(), N, layout)) for t in grads)
    for kvh in (0, Hkv - 1):
        heads = slice(kvh * group, (kvh + 1) * group)
        pairs = [t[:, kvh:kvh + 1].expand(-1, group, -1, -1) for t in (k, v)]
        want_q, want_k, want_v = hp.oracle_backward(q[:, heads], *pairs, only[:, heads], 1.0 / np.sqrt(d))
        hp.check_grad("dQ", dq[:, heads].numpy(), want_q, True)
        hp.check_grad("dK", dk[:, kvh:kvh + 1].numpy(), want_k.sum(1, keepdims=True), True)
        hp.check_grad("dV", dv[:, kvh:kvh + 1].numpy(), want_v.sum(1, keepdims=True), True)


@pytest.mark.parametrize("H,Hkv,c,d", [(204, 68, 384, 64), (490, 70, 384, 48), (213, 71, 300, 24), (142, 71, 193, 136)])
def test_groups_in_step_with_the_places_at_other_columns(H, Hkv, c, d):
    # (bwd_mfma.hip's launch of both kinds: every fourth, eighth, fourth and, with two workgroups a key tile, second owns keys)
    a = routes.args(c, d, H, Hkv)
    assert routes.backward(a) == "128 rows" and routes.one_launch(a)
    step_against_the_oracle(1, H, Hkv, c, d, 1, 0, sa.STRIPED)


@pytest.mark.parametrize("side", ["stride_s", "kv_stride_s"])
@pytest.mark.parametrize("c,d", [(128, 128), (250, 100)])
def test_rows_at_the_end_of_reach(c, d, side):
    # the rows of one side (rounded up to a tile) end just below 2^31 bytes; three requests lie behind the last tile
    pitch = (1 << 31) // (2 * ((c + 127) // 128 * 128)) - 64
    a = routes.args(c, d, 1, q_dev=0, layout=sa.CONTIGUOUS, **{side: pitch})
    assert routes.backward(a) == "128 rows" and routes.one_launch(a)
    x = [inputs.gaussian((1, 1, c, d), 30 + d + i, torch.bfloat16) for i in range(4)]
    want = hp.oracle_backward(*x, 1.0 / np.sqrt(d))
    o, want_lse = hp.oracle_forward(*x[:3], 1.0 / np.sqrt(d))
    wide = lambda dtype: torch.empty(c * pitch, dtype=dtype, device="cuda").as_strided((1, 1, c, d), (c * pitch, c * pitch, pitch, 1))  # noqa: E731
    f32 = dict(dtype=torch.float32, device="cuda")
    lse = torch.from_numpy(want_lse).to(**f32)
    q, k, v, g = (wide(t.dtype).copy_(t) if (i in (1, 2)) == (side == "kv_stride_s") else t.cuda() for i, t in enumerate(x))
    grads = [wide(torch.float32).zero_() if t.stride(2) == pitch else torch.zeros(1, 1, c, d, **f32) for t in (q, k, v)]
    delta = torch.from_numpy((inputs.to_f64(x[3]) * o).sum(-1)).to(**f32)
    sa.sa_attn_step_bwd(q, k, v, g, lse, delta, *grads, 0, 0, 1, sa.CONTIGUOUS, sa.shard_shape(q, c, lse, kv=k))
    torch.cuda.synchronize()
    for name, got, w in zip(("dQ", "dK", "dV"), grads, want):
        hp.check_grad(name, got.contiguous().cpu().numpy(), w, True)


def test_both_launches_give_the_same_bits():
    # 70 heads share one launch of both kinds, 280 do not: the order of the workgroups and the kernel of dQ touch no sum
    c, d = 250, 100
    assert routes.one_launch(routes.args(c, d, 70)) and not routes.one_launch(routes.args(c, d, 280))
    q, k, v, g = (inputs.gaussian((1, 280, c, d), 50 + i, torch.bfloat16).cuda() for i in range(4))
    lse, delta = torch.full((1, 280, c), 6.0, device="cuda"), inputs.gaussian((1, 280, c), 5).cuda()
    all_heads, halves = ([torch.zeros(1, 280, c, d, device="cuda") for _ in range(3)] for _ in range(2))
    sa.sa_attn_step_bwd(q, k, v, g, lse, delta, *all_heads, 1, 0, 2, sa.STRIPED, sa.shard_shape(q, c, lse))
    for h in range(0, 280, 70):
        part = [t[:, h:h + 70] for t in (q, k, v, g, lse, delta, *halves)]
        sa.sa_attn_step_bwd(*part, 1, 0, 2, sa.STRIPED, sa.shard_shape(part[0], c, part[4]))
    torch.cuda.synchronize()
    for a, b in zip(all_heads, halves):
        assert torch.equal(a, b)
