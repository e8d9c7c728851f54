"""bf16 blocks shorter than one 128-row tile run on the bf16 matrix cores in fp32 precision
(probabilities and dS as three bf16 terms).  Against the oracle with the fp32 configuration's bounds:
edges of the 32-row sub-tiles and of the second 64-row tile, partial 16-byte chunks, grouped heads,
the drivers' walk over several shards and single steps, on both sides of the forward's rule (more than
384 heads of up to 32 columns: a single block goes to the fp32 instruction)."""
import numpy as np
import pytest
import torch

from oracle import striped_attention as orc
from paper_2311_09431_amd import binding as sa
from paper_2311_09431_amd import inputs
from tests import helpers as hp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout", [sa.CONTIGUOUS, sa.STRIPED])
@pytest.mark.parametrize("H,Hkv,c,d,N", [
    (1, 1, 1, 4, 3), (2, 2, 31, 64, 2), (2, 1, 32, 36, 3), (1, 1, 64, 128, 4), (3, 3, 65, 100, 2),
    (4, 2, 97, 112, 2), (2, 2, 127, 128, 3), (40, 40, 64, 60, 2), (22, 11, 96, 124, 2),
    (384, 384, 40, 28, 2), (385, 385, 40, 32, 2), (513, 513, 20, 32, 2), (385, 385, 33, 36, 2),
])
@pytest.mark.parametrize("driver", [True, False])
def test_edges(layout, H, Hkv, c, d, N, driver):
    S, scale = N * c, 1.0 / np.sqrt(d)
    Q, dO = (inputs.gaussian((1, H, S, d), 11 + c + i, torch.bfloat16) for i in (0, 1))
    K, V = (inputs.gaussian((1, Hkv, S, d), 21 + c + i, torch.bfloat16) for i in (0, 1))
    Qp, Kp, Vp, dOp = (hp.to_device_order(x.cuda(), N, layout) for x in (Q, K, V, dO))
    f32 = dict(dtype=torch.float32, device="cuda")
    O, LSE = torch.empty(1, H, S, d, **f32), torch.empty(1, H, S, **f32)
    delta, (dQ, dK, dV) = torch.empty_like(LSE), [torch.zeros(x.shape, **f32) for x in (Qp, Kp, Vp)]
    shape = sa.shard_shape(Qp, c, LSE, kv=Kp if Hkv != H else None)
    sa.sa_ring_fwd(Qp, Kp, Vp, O, LSE, N, layout, shape, timed=not driver)       # timed: block by block
    sa.sa_ring_bwd(Qp, Kp, Vp, dOp, O, LSE, delta, dQ, dK, dV, N, layout, shape, timed=not driver)
    torch.cuda.synchronize()
    group = H // Hkv
    # every head on small cases, the first and the last ones of the many-head ones
    if H > 40:
        assert H == Hkv
        pick = lambda t: t[:, [0, H - 1]]                                          # noqa: E731
        Q, K, V, dO, O, LSE, dQ, dK, dV = (pick(t) for t in (Q, K, V, dO, O, LSE, dQ, dK, dV))
        Hkv = 2
    q, g = inputs.to_f64(Q), inputs.to_f64(dO)
    k, v = (np.repeat(inputs.to_f64(x), group, axis=1) for x in (K, V))
    host = lambda t: hp.from_device_order_host(t.cpu().numpy(), N, layout)
    Ow, Lw = orc.causal_attention_bh(q, k, v, scale)
    dQw, dKw, dVw = orc.causal_attention_grad_bh(q, k, v, g, scale)
    fold = lambda x: x.reshape(1, Hkv, group, S, d).sum(axis=2)
    assert hp.max_abs_err(host(O), Ow) <= 1e-5 and hp.max_abs_err(host(LSE), Lw) <= 1e-5
    for name, got, want in zip(("dQ", "dK", "dV"), (dQ, dK, dV), (dQw, fold(dKw), fold(dVw))):
        hp.check_grad(name, host(got), want, False)
