"""Backward steps on both sides of the rules that choose the split of the work: 32-row workgroups
(few rows), both kinds of 128-row workgroups in one launch, one launch each.  Against the oracle at
the edges of the tiles: blocks of exactly one tile, one row more, a last tile of one row, partial
16-byte chunks, grouped heads, triangular (both offsets) and full blocks."""
import numpy as np
import pytest
import torch

from paper_2311_09431_amd import binding as sa
from paper_2311_09431_amd import inputs
from tests import helpers as hp
from tests import routes

pytestmark = pytest.mark.gpu

CASES = [
    # B, H, H_kv, c, d: 128-row tiles of the key-owning side
    (1, 1, 1, 128, 128),        # 1
    (1, 2, 2, 129, 64),         # 4
    (1, 3, 3, 257, 100),        # 9, last tile of one row
    (2, 2, 1, 384, 112),        # 6, grouped heads
    (1, 16, 16, 512, 36),       # 64: split
    (1, 13, 13, 640, 128),      # 65: short walks, 128 rows
    (1, 32, 4, 256, 128),       # 8, 32 query heads
    (1, 8, 8, 512, 100),        # 32
    (1, 9, 9, 500, 100),        # 36
    (1, 64, 64, 512, 64),       # 256: one launch of 128-row workgroups for uneven work, not for full blocks
    (1, 43, 43, 768, 128),      # 258: one launch each
    (1, 24, 24, 520, 256),      # two key-owning workgroups per tile: 240 of 512
    (1, 3, 3, 130, 200),
]


@pytest.mark.parametrize("q_dev,kv_dev,layout", [(1, 0, sa.STRIPED), (0, 1, sa.STRIPED), (1, 0, sa.CONTIGUOUS)])
@pytest.mark.parametrize("B,H,Hkv,c,d", CASES)
def test_step_against_the_oracle(B, H, Hkv, c, d, q_dev, kv_dev, layout):
    # one block, softmax over the block alone (LSE and delta of it), two heads checked
    scale, dt = 1.0 / np.sqrt(d), torch.bfloat16
    q, g = (inputs.gaussian((B, H, c, d), 60 + c + i, dt) for i in (0, 1))
    k, v = (inputs.gaussian((B, Hkv, c, d), 70 + c + i, dt) for i in (0, 1))
    a, b = np.arange(c)[:, None], np.arange(c)[None, :]
    allowed = (b <= a - (kv_dev > q_dev)) if layout == sa.STRIPED or q_dev == kv_dev else np.ones((c, c), bool)
    gq, gg, gk, gv = (x.cuda() for x in (q, g, k, v))
    f32 = dict(dtype=torch.float32, device="cuda")
    o, lse, delta = torch.empty(B, H, c, d, **f32), torch.empty(B, H, c, **f32), torch.empty(B, H, c, **f32)
    dq, dk, dv = torch.zeros(B, H, c, d, **f32), torch.zeros(B, Hkv, c, d, **f32), torch.zeros(B, Hkv, c, d, **f32)
    shape = sa.shard_shape(gq, c, lse, kv=gk if Hkv != H else None)
    sa.sa_state_init(o, lse, shape)
    sa.sa_attn_step_fwd(gq, gk, gv, o, lse, q_dev, kv_dev, 2, layout, shape)
    # a row without a key has LSE = -inf and no P; any finite LSE stands for it
    lse = torch.where(torch.isinf(lse), torch.zeros_like(lse), lse)
    sa.sa_bwd_preprocess(o, gg, delta, shape)
    sa.sa_attn_step_bwd(gq, gk, gv, gg, lse, delta, dq, dk, dv, q_dev, kv_dev, 2, layout, shape)
    torch.cuda.synchronize()
    group = H // Hkv
    for kvh in {0, Hkv - 1}:
        wk, wv = np.zeros((c, d)), np.zeros((c, d))
        for h in range(kvh * group, (kvh + 1) * group):
            x = {n: inputs.to_f64(t[B - 1, i]) for n, t, i in (("q", q, h), ("g", g, h), ("k", k, kvh), ("v", v, kvh))}
            s = np.where(allowed, x["q"] @ x["k"].T * scale, -np.inf)
            p = np.exp(s - np.where(allowed.any(1), s.max(1, initial=-np.inf, where=allowed), 0.0)[:, None])
            p /= np.maximum(p.sum(1, keepdims=True), 1e-300)
            dp = x["g"] @ x["v"].T
            ds = p * (dp - (p * dp).sum(1, keepdims=True))
            wk += scale * ds.T @ x["q"]
            wv += p.T @ x["g"]
            hp.check_grad("dQ", dq[B - 1, h].cpu().numpy(), scale * ds @ x["k"], True)
        hp.check_grad("dK", dk[B - 1, kvh].cpu().numpy(), wk, True)
        hp.check_grad("dV", dv[B - 1, kvh].cpu().numpy(), wv, True)


@pytest.mark.parametrize("c,d,route", [(128, 128, "128 rows"), (250, 60, "128 rows"), (120, 100, "fp32")])
def test_rows_at_the_end_of_reach(c, d, route):
    # K, V, dK, dV rows so far apart that the block's rows (rounded up to a tile) just end below 2^31 bytes, but not the
    # rows behind them that the split kernels' last requests name
    pitch = (1 << 31) // (2 * ((c + 127) // 128 * 128)) - 64
    a = routes.args(c, d, 1, q_dev=0, layout=sa.CONTIGUOUS, kv_stride_s=pitch)
    assert routes.forward(a) == routes.backward(a) == route
    wide = lambda dtype: torch.empty(c * pitch, dtype=dtype, device="cuda").as_strided((1, 1, c, d), (c * pitch, c * pitch, pitch, 1))  # noqa: E731
    q, g, k0, v0 = (inputs.gaussian((1, 1, c, d), 30 + d + i, torch.bfloat16) for i in range(4))
    gq, gg, k, v, dk, dv = q.cuda(), g.cuda(), wide(q.dtype), wide(q.dtype), wide(torch.float32), wide(torch.float32)
    k.copy_(k0), v.copy_(v0), dk.zero_(), dv.zero_()
    f32 = dict(dtype=torch.float32, device="cuda")
    o, lse, delta, dq = (torch.zeros(*s, **f32) for s in ((1, 1, c, d), (1, 1, c), (1, 1, c), (1, 1, c, d)))
    shape = sa.shard_shape(gq, c, lse, kv=k)
    sa.sa_state_init(o, lse, shape)
    sa.sa_attn_step_fwd(gq, k, v, o, lse, 0, 0, 1, sa.CONTIGUOUS, shape)
    sa.sa_bwd_preprocess(o, gg, delta, shape)
    sa.sa_attn_step_bwd(gq, k, v, gg, lse, delta, dq, dk, dv, 0, 0, 1, sa.CONTIGUOUS, shape)
    torch.cuda.synchronize()
    want_o, want_l = hp.oracle_forward(q, k0, v0, 1.0 / np.sqrt(d))
    assert hp.max_abs_err(o.cpu().numpy(), want_o) <= 2e-2 and hp.max_abs_err(lse.cpu().numpy(), want_l) <= 1e-3
    for name, got, want in zip(("dQ", "dK", "dV"), (dq, dk, dv), hp.oracle_backward(q, k0, v0, g, 1.0 / np.sqrt(d))):
        hp.check_grad(name, got.contiguous().cpu().numpy(), want, True)


SPLIT = [
    # B, H, H_kv, c, d: more than 64 key tiles, long walks
    (1, 20, 20, 513, 64),       # 100; 340 workgroups of a kind, an uneven number of units of 8
    (2, 7, 7, 1500, 36),        # 168 (triangular only), ranks in chunks of four and three left over
    (1, 29, 29, 1100, 64),      # 261 (triangular only), an odd number of heads: chunks of eight ranks
    (1, 24, 12, 1300, 60),      # 132 (triangular only), grouped heads
    (1, 7, 7, 2100, 100),       # 119 (triangular only)
    (1, 32, 8, 1030, 128),      # 72, four heads per key/value head
    (1, 104, 13, 640, 72),      # 65, eight heads per key/value head, ranks in chunks of eight and four left over
    (1, 110, 55, 384, 64),      # 165 (triangular only), few ranks: in chunks all the same
]


@pytest.mark.parametrize("q_dev,kv_dev,layout", [(1, 0, sa.STRIPED), (0, 1, sa.STRIPED), (1, 0, sa.CONTIGUOUS)])
@pytest.mark.parametrize("B,H,Hkv,c,d", SPLIT)
def test_larger_split_launches(B, H, Hkv, c, d, q_dev, kv_dev, layout):
    a = routes.args(c, d, H, Hkv, B, q_dev=q_dev, kv_dev=kv_dev, layout=layout)
    full = layout == sa.CONTIGUOUS
    assert routes.backward(a) == ("128 rows" if full and c not in (513, 1030, 640) else "split")
    if not full:
        test_step_against_the_oracle(B, H, Hkv, c, d, q_dev, kv_dev, layout)
    if routes.backward(a) != "split":
        return
    # every head as a launch of its own gives it: the order of a launch's workgroups touches no sum
    q, g = (inputs.gaussian((B, H, c, d), 60 + c + i, torch.bfloat16).cuda() for i in (0, 1))
    k, v = (inputs.gaussian((B, Hkv, c, d), 70 + c + i, torch.bfloat16).cuda() for i in (0, 1))
    f32 = dict(dtype=torch.float32, device="cuda")
    lse, delta = torch.full((B, H, c), 7.0, **f32), inputs.gaussian((B, H, c), 5).cuda()
    whole, single = ([torch.zeros(x.shape, **f32) for x in (q, k, v)] for _ in range(2))
    group = H // Hkv
    sa.sa_attn_step_bwd(q, k, v, g, lse, delta, *whole, q_dev, kv_dev, 2, layout, sa.shard_shape(q, c, lse, kv=k))
    for b in range(B):
        for h in range(Hkv):
            own = slice(h * group, (h + 1) * group)
            sq, sg, sl, sd, sdq = (x[b:b + 1, own] for x in (q, g, lse, delta, single[0]))
            sk, sv, sdk, sdv = (x[b:b + 1, h:h + 1] for x in (k, v, *single[1:]))
            sa.sa_attn_step_bwd(sq, sk, sv, sg, sl, sd, sdq, sdk, sdv, q_dev, kv_dev, 2, layout, sa.shard_shape(sq, c, sl, kv=sk))
    torch.cuda.synchronize()
    for x, y in zip(whole, single):
        assert torch.equal(x, y)
