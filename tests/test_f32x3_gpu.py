"""fp32 launches that fill the chip run on the bf16 matrix cores with every operand as three bf16
terms, in workgroups of 128 rows (forward of 512 such tiles and more: 256).  Against the oracle at the edges of their
32-row tiles and workgroups, at the forward's line, with grouped heads and with scores that spread over many powers of
two; the bounds are the fp32 configuration's."""
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
    # B, H, H_kv, c, d, N, spread of q and k; the directions these kernels take
    (1, 96, 96, 17, 4, 1, 1.0, "fb"),           # half a tile
    (2, 128, 128, 33, 36, 1, 1.0, "fb"),        # half a chunk, a tile of one row
    (2, 64, 64, 129, 64, 1, 1.0, "fb"),         # last workgroup of one row
    (4, 32, 8, 129, 64, 2, 1.0, "f"),           # grouped heads
    (2, 32, 32, 260, 100, 2, 1.0, "fb"),
    (1, 64, 64, 256, 128, 1, 1.0, "fb"),        # 128 row tiles: four-wave workgroups
    (1, 64, 64, 300, 128, 3, 2.0, "fb"),        # 576: eight
    (1, 200, 50, 300, 36, 1, 1.0, "fb"),
    (4, 64, 64, 1, 4, 2, 1.0, ""),              # (few rows or tiles: other kernels)
    (4, 64, 64, 33, 36, 2, 1.0, ""),
    (1, 43, 43, 256, 128, 3, 1.0, "b"),
    (1, 32, 2, 260, 36, 3, 1.0, ""),
    (4, 16, 4, 300, 36, 3, 1.0, "f"),
]


@pytest.mark.parametrize("layout", [sa.CONTIGUOUS, sa.STRIPED])
@pytest.mark.parametrize("B,H,Hkv,c,d,N,std,these", CASES)
def test_edges(layout, B, H, Hkv, c, d, N, std, these):
    for back in (False, True):
        if "fb"[back] in these:
            assert routes.f32(routes.args(c, d, H, Hkv, B=B, layout=layout, N=N), back).startswith("128 rows")
    S, scale = N * c, 1.0 / np.sqrt(d)
    Q = inputs.gaussian((B, H, S, d), c + d, torch.float32, std)
    K = inputs.gaussian((B, Hkv, S, d), c + d + 1, torch.float32, std)
    V = inputs.gaussian((B, Hkv, S, d), c + d + 2)
    dO = inputs.gaussian((B, H, S, d), c + d + 3)
    Qp, Kp, Vp, dOp = (hp.to_device_order(x.cuda(), N, layout) for x in (Q, K, V, dO))
    f32 = dict(dtype=torch.float32, device="cuda")
    O, LSE = torch.empty(B, H, S, d, **f32), torch.empty(B, H, S, **f32)
    delta, grads = torch.empty_like(LSE), [torch.empty_like(x) for x in (Qp, Kp, Vp)]
    shape = sa.shard_shape(Qp, c, LSE, kv=Kp if Hkv != H else None)
    sa.sa_ring_fwd(Qp, Kp, Vp, O, LSE, N, layout, shape)
    sa.sa_ring_bwd(Qp, Kp, Vp, dOp, O, LSE, delta, *grads, N, layout, shape)
    torch.cuda.synchronize()
    group = H // Hkv
    for b, kvh in {(0, 0), (B - 1, Hkv - 1)}:          # first and last group of heads
        hs = slice(kvh * group, (kvh + 1) * group)
        q, g = (inputs.to_f64(x[b:b + 1, hs]) for x in (Q, dO))
        k, v = (np.repeat(inputs.to_f64(x[b:b + 1, kvh:kvh + 1]), group, axis=1) for x in (K, V))
        Ow, Lw = orc.causal_attention_bh(q, k, v, scale)
        dQw, dKw, dVw = orc.causal_attention_grad_bh(q, k, v, g, scale)
        host = lambda t, sel: hp.from_device_order_host(t[b:b + 1, sel].cpu().numpy(), N, layout)
        assert hp.max_abs_err(host(O, hs), Ow) <= 1e-5
        assert hp.max_abs_err(host(LSE, hs), Lw) <= 1e-5
        hp.check_grad("dQ", host(grads[0], hs), dQw, False)
        one = slice(kvh, kvh + 1)
        hp.check_grad("dK", host(grads[1], one), dKw.sum(axis=1, keepdims=True), False)
        hp.check_grad("dV", host(grads[2], one), dVw.sum(axis=1, keepdims=True), False)


def test_a_score_of_minus_infinity_is_no_key():
    # an infinite key element makes scores of +-inf; where the row's query keeps them at -inf the key
    # drops out, as with the fp32 instruction
    B, H, c, d = 4, 64, 40, 32
    assert routes.f32(routes.args(c, d, H, B=B), False) == "128 rows"
    Q, K, V = (inputs.gaussian((B, H, c, d), 5 + i).cuda() for i in range(3))
    Q[..., 0] = Q[..., 0].abs() + 0.1
    K[:, :, 7, 0] = -float("inf")
    O, LSE = torch.empty_like(Q), torch.empty(B, H, c, device="cuda")
    shape = sa.shard_shape(Q, c, LSE)
    sa.sa_ring_fwd(Q, K, V, O, LSE, 1, sa.CONTIGUOUS, shape)
    K2 = K.double()
    s = (Q.double() @ K2.transpose(-1, -2).contiguous()) / d ** 0.5
    s = s.masked_fill(~torch.ones(c, c, dtype=torch.bool, device="cuda").tril(), -float("inf"))
    assert (O.double() - s.softmax(-1) @ V.double()).abs().max().item() <= 1e-5
    assert (LSE.double() - s.logsumexp(-1)).abs().max().item() <= 1e-5
