"""Forward launches on both sides of the rule that chooses the split of the work: 32-row workgroups whose
wavefronts share the keys (few rows) or 128-row ones.  Against the oracle at the edges of the tiles: blocks
of exactly one tile, a last sub-tile of one row, fewer sub-tiles than wavefronts, partial 16-byte chunks,
grouped heads; rings (many shards a walk) and a walk step by step, both layouts."""
import numpy as np
import pytest
import torch

from oracle import striped_attention as orc
from paper_2311_09431_amd import binding as sa
from paper_2311_09431_amd import inputs
from tests import helpers as hp
from tests import routes

pytestmark = pytest.mark.gpu

CASES = [
    # B, H, H_kv, c, d, N: 128-row tiles of all devices' queries (single steps: of one device's)
    (1, 1, 1, 128, 128, 1),         # one block of one tile
    (1, 1, 1, 128, 64, 1),          # (stays with a 128-row tile)
    (1, 2, 2, 129, 64, 2),          # 8, last sub-tile of one row
    (1, 2, 1, 162, 100, 3),         # 12, grouped heads, partial chunks
    (2, 2, 2, 254, 36, 2),          # 16
    (1, 8, 2, 1024, 128, 1),        # 64
    (1, 5, 5, 1664, 128, 1),        # 65, walk of more than 1024 keys
    (1, 26, 26, 600, 112, 1),       # 130
    (1, 16, 16, 384, 64, 2),        # 96
    (1, 2, 2, 2048, 64, 8),         # 256, long walk
]


@pytest.mark.parametrize("layout", [sa.STRIPED, sa.CONTIGUOUS])
@pytest.mark.parametrize("B,H,Hkv,c,d,N", CASES)
def test_rings_against_the_oracle(B, H, Hkv, c, d, N, layout):
    dt, S, group = torch.bfloat16, N * c, H // Hkv
    q = inputs.gaussian((B, H, S, d), 80 + c, dt)
    k, v = (inputs.gaussian((B, Hkv, S, d), 90 + c + i, dt) for i in (0, 1))
    gq, gk, gv = (hp.to_device_order(x.cuda(), N, layout) for x in (q, k, v))
    f32 = dict(dtype=torch.float32, device="cuda")
    outs = []
    for driver in (True, False):
        o, lse = torch.full((B, H, S, d), 7.0, **f32), torch.full((B, H, S), 7.0, **f32)
        shape = sa.shard_shape(gq, c, lse, kv=gk if Hkv != H else None)
        if driver:
            sa.sa_ring_fwd(gq, gk, gv, o, lse, N, layout, shape)
        else:
            rows = lambda x, i: x[:, :, i * c:]                       # noqa: E731
            for j in range(N):
                sa.sa_state_init(rows(o, j), rows(lse, j), shape)
            for _, j, i in orc.ring_schedule(N):
                sa.sa_attn_step_fwd(rows(gq, j), rows(gk, i), rows(gv, i), rows(o, j), rows(lse, j), j, i, N, layout, shape)
        outs.append((o, lse))
    torch.cuda.synchronize()
    for h in {0, H - 1}:
        want_o, want_l = hp.oracle_forward(q[B - 1:, h:h + 1], k[B - 1:, h // group:h // group + 1],
                                           v[B - 1:, h // group:h // group + 1], 1.0 / np.sqrt(d))
        for o, lse in outs:
            got_o, got_l = (hp.from_device_order_host(x[B - 1:, h:h + 1].cpu().numpy(), N, layout) for x in (o, lse))
            # P is rounded to bf16 (2^-9 of each term) before its product, as everywhere in bf16
            assert hp.max_abs_err(got_o, want_o) <= 2e-2
            assert np.linalg.norm(got_o - want_o) <= 4e-3 * np.linalg.norm(want_o)
            assert hp.max_abs_err(got_l, want_l) <= 1e-3


@pytest.mark.parametrize("c,H,d,shape_n,route", [
    (256, 2, 64, 2, "split"), (640, 13, 128, 1, "split"), (512, 32, 64, 1, "split"), (512, 33, 64, 2, "128 rows"),
    (640, 27, 128, 2, "128 rows"),
])
def test_fused_rotation_like_rotated_queries(c, H, d, shape_n, route):
    # on both sides of the rule; the two sine evaluations round a few queries to neighbouring bf16 values
    assert routes.forward(routes.args(c, d, H, B=shape_n)) == route
    dt, f32 = torch.bfloat16, dict(dtype=torch.float32, device="cuda")
    q, k, v = (inputs.gaussian((shape_n, H, c, d), 100 + i, dt).cuda() for i in range(3))
    pos = (torch.arange(c, dtype=torch.int32) * 8 + 1).cuda()
    o, lse = ([torch.empty(s, **f32) for _ in range(2)] for s in ((shape_n, H, c, d), (shape_n, H, c)))
    shape = sa.shard_shape(q, c, lse[0])
    for i in range(2):
        sa.sa_state_init(o[i], lse[i], shape)
    sa.sa_attn_step_fwd_rope(q, k, v, o[0], lse[0], pos, 1, 0, 8, sa.STRIPED, shape)
    qr = torch.empty_like(q)
    sa.sa_rope(q, qr, pos, shape)
    sa.sa_attn_step_fwd(qr, k, v, o[1], lse[1], 1, 0, 8, sa.STRIPED, shape)
    assert float((o[0] - o[1]).norm() / o[1].norm()) <= 1e-3
    assert hp.max_abs_err(lse[0].cpu().numpy(), lse[1].cpu().numpy()) <= 5e-3


@pytest.mark.parametrize("c,d,pitch,fused", [
    (128, 128, 1 << 24, False), (160, 100, 1 << 23, False), (8192, 64, (1 << 18) + 8, False), (128, 128, 1 << 24, True),
    (8192, 64, (1 << 18) + 8, True),
])
def test_query_rows_far_apart(c, d, pitch, fused):
    # Q (and O) narrow views of a wide buffer, K and V packed: 4 GiB and more, or between 2 and 4, from the first to
    # the last row of a launch small enough for the split kernel, whose offsets have 32 bits.  NaN behind every row.
    assert routes.forward(routes.args(c, d, 1, q_dev=0, layout=sa.CONTIGUOUS, stride_s=pitch)) == "128 rows"
    f32, bf = dict(dtype=torch.float32, device="cuda"), dict(dtype=torch.bfloat16, device="cuda")
    wide = lambda **kw: torch.empty((c - 1) * pitch + d + 64, **kw).as_strided((1, 1, c, d + 64), (c * pitch, c * pitch, pitch, 1))  # noqa: E731
    q, k, v = (inputs.gaussian((1, 1, c, d), 20 + i, torch.bfloat16).cuda() for i in range(3))
    qw, ow = wide(**bf).fill_(float("nan"))[..., :d], wide(**f32)[..., :d]
    qw.copy_(q)
    pos = torch.arange(c, dtype=torch.int32, device="cuda") * 3
    outs = []
    for x, o in ((qw, ow), (q, torch.empty(1, 1, c, d, **f32))):
        lse = torch.empty(1, 1, c, **f32)
        shape = sa.shard_shape(x, c, lse, kv=k)
        sa.sa_state_init(o, lse, shape)
        if fused:
            sa.sa_attn_step_fwd_rope(x, k, v, o, lse, pos, 0, 0, 1, sa.CONTIGUOUS, shape)
        else:
            sa.sa_attn_step_fwd(x, k, v, o, lse, 0, 0, 1, sa.CONTIGUOUS, shape)
        outs.append((o.contiguous(), lse))
    torch.cuda.synchronize()
    (o, lse), (o1, lse1) = outs
    # the packed call's kernel rounds P to bf16 against other references
    assert float((o - o1).norm()) <= 4e-3 * float(o1.norm())
    assert hp.max_abs_err(lse.cpu().numpy(), lse1.cpu().numpy()) <= 1e-3
    if not fused:
        want_o, want_l = hp.oracle_forward(q, k, v, 1.0 / np.sqrt(d))
        assert hp.max_abs_err(o.cpu().numpy(), want_o) <= 2e-2
        assert hp.max_abs_err(lse.cpu().numpy(), want_l) <= 1e-3
