"""The ring drivers fold all blocks of a device into one walk (no per-step timings asked for); the
step entry points and the timed drivers run block by block.  Both against the oracle, at the edges
of the walk: blocks of one tile pair, a single device, ragged blocks, grouped heads, the last shard
of the contiguous layout, and the parts of dQ / dK / dV that one device's share does not touch."""
import numpy as np
import pytest
import torch

from oracle import striped_attention as orc
from paper_2311_09431_amd import binding as sa
from paper_2311_09431_amd import inputs
from tests import helpers as hp

pytestmark = pytest.mark.gpu

CASES = [
    # H, H_kv, c, d, N, dtype
    (2, 2, 128, 128, 4, torch.bfloat16),       # one tile pair per block
    (1, 1, 256, 64, 1, torch.bfloat16),        # one device: a walk of one block
    (2, 1, 200, 100, 3, torch.bfloat16),       # ragged, partial chunk, two heads per key/value head
    (2, 2, 384, 256, 3, torch.bfloat16),       # two column halves
    (4, 1, 40, 64, 3, torch.bfloat16),         # fp32 kernels
    (1, 1, 33, 32, 4, torch.float32),
    (2, 2, 160, 256, 2, torch.float32),
]


@pytest.mark.parametrize("layout", [sa.CONTIGUOUS, sa.STRIPED])
@pytest.mark.parametrize("H,Hkv,c,d,N,dtype", CASES)
def test_drivers_against_the_oracle(layout, H, Hkv, c, d, N, dtype):
    S, scale, bf16 = N * c, 1.0 / np.sqrt(d), dtype is torch.bfloat16
    Q, dO = (inputs.gaussian((1, H, S, d), 900 + c + i, dtype) for i in (0, 1))
    K, V = (inputs.gaussian((1, Hkv, S, d), 950 + c + i, dtype) for i in (0, 1))
    q, k, v, g = (inputs.to_f64(x) for x in (Q, K, V, dO))
    kr, vr = (np.repeat(x, H // Hkv, axis=1) for x in (k, v))
    Ow, Lw = orc.causal_attention_bh(q, kr, vr, scale)
    dQw, dKw, dVw = orc.causal_attention_grad_bh(q, kr, vr, g, scale)
    fold = lambda x: x.reshape(1, Hkv, H // Hkv, S, d).sum(axis=2)
    Qp, Kp, Vp, dOp = (hp.to_device_order(x.cuda(), N, layout) for x in (Q, K, V, dO))
    f32 = dict(dtype=torch.float32, device="cuda")
    LSE = torch.empty(1, H, S, **f32)
    shape = sa.shard_shape(Qp, c, LSE, kv=Kp if Hkv != H else None)
    host = lambda t: hp.from_device_order_host(t.cpu().numpy(), N, layout)

    def play(dev, timed):
        O, L, delta = torch.full_like(Qp, 7.0, dtype=torch.float32), torch.full_like(LSE, 7.0), torch.empty_like(LSE)
        grads = [torch.full_like(x, 7.0, dtype=torch.float32) for x in (Qp, Kp, Vp)]
        sa.sa_ring_fwd(Qp, Kp, Vp, O, L, N, layout, shape, dev, timed)
        sa.sa_ring_bwd(Qp, Kp, Vp, dOp, O, L, delta, *grads, N, layout, shape, dev, timed)
        torch.cuda.synchronize()
        return O, L, grads

    for timed in (False, True):
        O, L, grads = play(-1, timed)
        assert hp.max_abs_err(host(O), Ow) <= (2e-2 if bf16 else 1e-5)
        assert hp.max_abs_err(host(L), Lw) <= (1e-3 if bf16 else 1e-5)
        for name, got, want in zip(("dQ", "dK", "dV"), grads, (dQw, fold(dKw), fold(dVw))):
            hp.check_grad(name, host(got), want, bf16)
    # shares: the device's rows as in the whole ring, other rows of O untouched and of dQ zero,
    # the shares of dK and dV adding up to the whole
    whole_O, whole_L, whole = play(-1, False)
    sums = [torch.zeros_like(x) for x in whole[1:]]
    for dev in range(N):
        O, L, (dQ, dK, dV) = play(dev, False)
        own = slice(dev * c, (dev + 1) * c)
        others = [r for r in range(S) if not own.start <= r < own.stop]
        assert torch.equal(O[:, :, own], whole_O[:, :, own]) and torch.equal(L[:, :, own], whole_L[:, :, own])
        assert torch.equal(dQ[:, :, own], whole[0][:, :, own])
        assert bool((O[:, :, others] == 7.0).all()) and bool((dQ[:, :, others] == 0.0).all())
        if layout == sa.CONTIGUOUS:      # shards further on are not seen
            assert bool((dK[:, :, own.stop:] == 0.0).all()) and bool((dV[:, :, own.stop:] == 0.0).all())
        sums[0] += dK
        sums[1] += dV
    for name, got, want in zip(("dK", "dV"), sums, (fold(dKw), fold(dVw))):
        hp.check_grad(name, host(got), want, bf16)


@pytest.mark.parametrize("H,c,N,d", [(2, 256, 8, 64), (1, 512, 4, 128), (2, 200, 5, 100)])
def test_a_striped_walk_is_as_close_as_its_steps(H, c, N, d):
    # probabilities are rounded to bf16 against a reference; the largest of a row's first keys in a shard is 1,
    # exactly, and the first rows, which carry most of O's norm, have few others.  With one reference for all
    # shards the error of O was 1.25 to 1.5 times that of the steps.  1.02: the two fold the shards
    # in another order.
    S = N * c
    Q, K, V = (inputs.gaussian((1, H, S, d), 70 + c + i, torch.bfloat16) for i in range(3))
    want, _ = orc.causal_attention_bh(*(inputs.to_f64(x) for x in (Q, K, V)), 1.0 / np.sqrt(d))
    q, k, v = (hp.to_device_order(x.cuda(), N, sa.STRIPED) for x in (Q, K, V))
    O, LSE = torch.empty(1, H, S, d, device="cuda"), torch.empty(1, H, S, device="cuda")
    shape = sa.shard_shape(q, c, LSE)
    err = {}
    for timed in (False, True):
        sa.sa_ring_fwd(q, k, v, O, LSE, N, sa.STRIPED, shape, -1, timed)
        torch.cuda.synchronize()
        got = hp.from_device_order_host(O.cpu().numpy(), N, sa.STRIPED)
        err[timed] = np.linalg.norm(got - want)
    assert err[False] <= 1.02 * err[True], err
