"""Rings of many short shards over as many (batch, head) pairs as the entry points take: more
workgroups than one launch may hold (HIP: fewer than 2^32 threads), which the drivers play in parts.
One row a shard and 257 devices; a few heads against fp64, the last of a part and the first of the next
among them.  And fp32 steps of as many heads, whose kernels have up to 512 threads per 32 rows."""
import numpy as np
import pytest
import torch

from paper_2311_09431_amd import binding as sa
from paper_2311_09431_amd import inputs

pytestmark = pytest.mark.gpu

N, D, HEADS = 257, 4, 65535


def tensors(B, H, Hkv):
    t = {n: inputs.gaussian((B, h, N, D), 3 + i, torch.bfloat16, device="cuda")
         for i, (n, h) in enumerate((("q", H), ("k", Hkv), ("v", Hkv), ("g", H)))}
    f32 = dict(dtype=torch.float32, device="cuda")
    t.update(o=torch.empty(B, H, N, D, **f32), lse=torch.empty(B, H, N, **f32), delta=torch.empty(B, H, N, **f32),
             dq=torch.empty(B, H, N, D, **f32), dk=torch.empty(B, Hkv, N, D, **f32), dv=torch.empty(B, Hkv, N, D, **f32))
    return t, sa.shard_shape(t["q"], 1, t["lse"], kv=t["k"] if H != Hkv else None)


def attention(q, K, V, n):
    s = K[:n] @ q / np.sqrt(D)
    p = np.exp(s - s.max())
    return p / p.sum(), s.max() + np.log(p.sum())


@pytest.mark.parametrize("B,H,Hkv", [(1, HEADS, HEADS), (5, HEADS // 5, HEADS // 15)])
def test_ring_of_many_shards(B, H, Hkv):
    t, shape = tensors(B, H, Hkv)
    sa.sa_ring_fwd(t["q"], t["k"], t["v"], t["o"], t["lse"], N, sa.CONTIGUOUS, shape)
    # the last device's share: one query row per head, every shard's key rows
    sa.sa_ring_bwd(t["q"], t["k"], t["v"], t["g"], t["o"], t["lse"], t["delta"], t["dq"], t["dk"], t["dv"], N,
                   sa.CONTIGUOUS, shape, N - 1)
    torch.cuda.synchronize()
    group = H // Hkv
    for b in {0, B - 1}:
        for kvh in {0, 1, Hkv // 2, Hkv - 2, Hkv - 1}:
            K, V = (inputs.to_f64(t[n][b, kvh]) for n in ("k", "v"))
            dk, dv = np.zeros((N, D)), np.zeros((N, D))
            for h in range(kvh * group, (kvh + 1) * group):
                q, g = (inputs.to_f64(t[n][b, h]) for n in ("q", "g"))
                o, lse = (t[n][b, h].cpu().numpy() for n in ("o", "lse"))
                for a in range(N):
                    p, L = attention(q[a], K, V, a + 1)
                    assert np.abs(o[a] - p @ V[:a + 1]).max() <= 1e-5 and abs(lse[a] - L) <= 1e-5, (b, h, a)
                ds = p * (V @ g[-1] - (V @ g[-1]) @ p) / np.sqrt(D)       # the last row's
                dq = t["dq"][b, h].cpu().numpy()
                assert np.abs(dq[-1] - ds @ K).max() <= 2e-5 and not dq[:-1].any()
                dk, dv = dk + np.outer(ds, q[-1]), dv + np.outer(p, g[-1])
            assert np.abs(t["dk"][b, kvh].cpu().numpy() - dk).max() <= 2e-5
            assert np.abs(t["dv"][b, kvh].cpu().numpy() - dv).max() <= 2e-5


def test_fp32_step_of_long_blocks():
    # 65535 heads of 2080 rows: with 32 rows to a workgroup of 512 threads the backward would hold 1.016 * 2^32 threads
    c = 2080
    f32 = dict(dtype=torch.float32, device="cuda")
    q, k, v, g = (inputs.gaussian((1, HEADS, c, D), 21 + i, device="cuda") for i in range(4))
    o, dq, dk, dv = (torch.zeros(1, HEADS, c, D, **f32) for _ in range(4))
    lse, delta = (torch.empty(1, HEADS, c, **f32) for _ in range(2))
    shape = sa.shard_shape(q, c, lse)
    sa.sa_state_init(o, lse, shape)
    sa.sa_attn_step_fwd(q, k, v, o, lse, 0, 0, 1, sa.STRIPED, shape)
    sa.sa_bwd_preprocess(o, g, delta, shape)
    sa.sa_attn_step_bwd(q, k, v, g, lse, delta, dq, dk, dv, 0, 0, 1, sa.STRIPED, shape)
    torch.cuda.synchronize()
    for h in (0, 1, HEADS // 2, HEADS - 1):
        Q, K, V, G = (inputs.to_f64(x[0, h]) for x in (q, k, v, g))
        s = np.where(np.tri(c, dtype=bool), Q @ K.T / np.sqrt(D), -np.inf)
        p = np.exp(s - s.max(axis=1, keepdims=True))
        p /= p.sum(axis=1, keepdims=True)
        ds = p * (G @ V.T - (p * (G @ V.T)).sum(axis=1, keepdims=True)) / np.sqrt(D)
        assert np.abs(o[0, h].cpu().numpy() - p @ V).max() <= 1e-5
        for got, want in ((dq, ds @ K), (dk, ds.T @ Q), (dv, p.T @ G)):
            assert np.abs(got[0, h].cpu().numpy() - want).max() <= 2e-5 * max(1.0, np.abs(want).max())
