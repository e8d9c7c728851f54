"""fp32 storage of up to 128 columns on the two kinds of kernels that only few launches take: short walks on the fp32
instruction, and in the backward one wavefront to 32 rows of the 128-row workgroups.  Against fp64 over the allowed
pairs, with grouped heads, infinities and NaN; the bounds are the fp32 configuration's.  And one device's share of a
ring against three shards and more by the 128-row kernels, whose query-owning workgroups then come first."""
import numpy as np
import pytest
import torch

from oracle import striped_attention as orc
from paper_2311_09431_amd import binding as sa
from paper_2311_09431_amd import inputs
from tests import helpers as hp
from tests import routes
from tests import test_nonfinite_gpu as nf

pytestmark = [pytest.mark.gpu, nf.np_quiet]

F32 = torch.float32
INSTRUCTION = [
    # H, H_kv, c, d, dtype
    (2, 2, 97, 128, F32),           # less than a round of four wavefronts
    (2, 1, 128, 116, F32),          # one round, a chunk of four columns
    (64, 64, 200, 32, F32),         # two, several workgroups to a compute unit
]
ALONE = [
    (130, 130, 128, 128, F32),      # one tile
    (130, 65, 129, 100, F32),       # a second one of one row, grouped heads
    (256, 256, 40, 72, F32),
]


@pytest.mark.parametrize("block", nf.BLOCKS[:2])
@pytest.mark.parametrize("route", INSTRUCTION)
def test_fp32_instruction(route, block):
    H, Hkv, c, d, _ = route
    for back in (False, True):
        assert routes.f32(routes.args(c, d, H, Hkv), back) == "fp32 instruction"
    nf.check_forward_step(route, block, lambda t, at: {"clean": lambda x: None, **nf.swallowed(t, at), **nf.masked(t, at)})
    nf.check_backward_step(route, block, lambda t, at: {"clean": lambda x: None, **nf.backward_kinds(t, at)})


@pytest.mark.parametrize("block", nf.BLOCKS[:2])
@pytest.mark.parametrize("route", ALONE)
def test_one_wavefront_to_32_rows(route, block):
    H, Hkv, c, d, _ = route
    assert routes.f32(routes.args(c, d, H, Hkv), True) == "128 rows, one wavefront"
    nf.check_backward_step(route, block, lambda t, at: {"clean": lambda x: None, **nf.backward_kinds(t, at)})


@pytest.mark.parametrize("layout", [sa.CONTIGUOUS, sa.STRIPED])
@pytest.mark.parametrize("N,H,c,d", [(3, 64, 300, 128), (4, 64, 260, 100), (3, 128, 130, 64)])
def test_one_device_against_many_shards(layout, N, H, c, d):
    S, dev, scale = N * c, N - 1, 1.0 / np.sqrt(d)
    a = routes.args(c, d, H, layout=layout, N=N)
    a.n_q, a.q_dev = 1, dev
    assert routes.f32(a, True) == "128 rows" and 2 * a.n_q < a.n_kv        # queries first
    Q, K, V, G = (inputs.gaussian((1, H, S, d), c + d + i) for i in range(4))
    q, k, v, g = (hp.to_device_order(x.cuda(), N, layout) for x in (Q, K, V, G))
    O, LSE = torch.empty_like(q), torch.empty(1, H, S, device="cuda")
    delta, grads = torch.empty_like(LSE), [torch.empty_like(q) for _ in range(3)]
    shape = sa.shard_shape(q, c, LSE)
    sa.sa_ring_fwd(q, k, v, O, LSE, N, layout, shape, dev)
    sa.sa_ring_bwd(q, k, v, g, O, LSE, delta, *grads, N, layout, shape, dev)
    torch.cuda.synchronize()
    rows = np.arange(dev, S, N) if layout == sa.STRIPED else np.arange(dev * c, S)
    for h in (0, H - 1):
        one = lambda x: inputs.to_f64(x[:, h:h + 1])        # noqa: E731
        Gd = np.zeros((1, 1, S, d))                         # the other devices' rows give nothing to dK and dV
        Gd[:, :, rows] = one(G)[:, :, rows]
        host = lambda x: hp.from_device_order_host(x[:, h:h + 1].cpu().numpy(), N, layout)      # noqa: E731
        Ow, Lw = orc.causal_attention_bh(one(Q), one(K), one(V), scale)
        assert hp.max_abs_err(host(O)[:, :, rows], Ow[:, :, rows]) <= 1e-5
        assert hp.max_abs_err(host(LSE)[:, :, rows], Lw[:, :, rows]) <= 1e-5
        for name, got, want in zip(("dQ", "dK", "dV"), grads, orc.causal_attention_grad_bh(one(Q), one(K), one(V), Gd, scale)):
            hp.check_grad(name, host(got), want, False)
