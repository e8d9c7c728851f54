"""The backward kernels with a ring of tiles (65 to 128 columns): walks of one tile and of few, last tiles of one row, partial
16-byte chunks, groups of heads, several shards in one walk, both kinds in one launch and each in its own."""
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
    # B, H, H_kv, c, d
    (1, 140, 140, 128, 128),        # one launch of both kinds for uneven work: walks of two tiles
    (1, 70, 70, 129, 100),          # ... a last tile of one row: a walk of one tile
    (2, 13, 13, 321, 68),           # ... 78 tiles, 65 rows behind the last whole one
    (1, 160, 40, 200, 112),         # ... four query heads in a walk
    (1, 130, 130, 257, 124),        # one launch each, the keys by ranks for uneven work
    (1, 800, 400, 128, 72),         # ... two query heads in a walk
]


@pytest.mark.parametrize("q_dev,kv_dev,layout", [(1, 0, sa.STRIPED), (0, 1, sa.STRIPED), (1, 0, sa.CONTIGUOUS), (1, 1, sa.CONTIGUOUS)])
@pytest.mark.parametrize("B,H,Hkv,c,d", STEPS)
def test_steps(B, H, Hkv, c, d, q_dev, kv_dev, layout):
    assert routes.backward(routes.args(c, d, H, Hkv, B, q_dev=q_dev, kv_dev=kv_dev, layout=layout)) == "128 rows"
    if q_dev == kv_dev:         # (the same mask as the striped layout's)
        layout, q_dev, kv_dev = sa.STRIPED, 1, 0
    step_against_the_oracle(B, H, Hkv, c, d, q_dev, kv_dev, layout)


@pytest.mark.parametrize("layout", [sa.STRIPED, sa.CONTIGUOUS])
@pytest.mark.parametrize("H,N,c,d,dev", [(24, 3, 200, 96, -1), (24, 3, 200, 96, 1), (70, 3, 192, 128, -1), (18, 4, 129, 100, 3)])
def test_walks_over_several_shards(H, N, c, d, dev, layout):
    S = N * c
    q, k, v, g = (inputs.gaussian((1, H, S, d), 40 + d + i, torch.bfloat16) for i in range(4))
    x = [hp.to_device_order(t.cuda(), N, layout) for t in (q, k, v, g)]
    o, lse = torch.empty(1, H, S, d, device="cuda"), torch.empty(1, H, S, device="cuda")
    shape = sa.shard_shape(x[0], c, lse)
    sa.sa_ring_fwd(*x[:3], o, lse, N, layout, shape)
    delta, grads = torch.empty_like(lse), [torch.full_like(o, float("nan")) for _ in range(3)]
    own = slice(dev * c, (dev + 1) * c) if dev >= 0 else slice(0, S)
    sa.sa_ring_bwd(*x, o, lse, delta, *grads, N, layout, shape, dev)
    torch.cuda.synchronize()
    # one device's part: dO of its own rows alone
    only = torch.zeros_like(x[3])
    only[:, :, own] = x[3][:, :, own]
    only = torch.from_numpy(hp.from_device_order_host(only.float().cpu().numpy(), N, layout)).to(torch.bfloat16)
    want = hp.oracle_backward(*hp.some_heads(q, k, v, only), 1.0 / np.sqrt(d))
    for name, got, w in zip(("dQ", "dK", "dV"), grads, want):
        got = hp.some_heads(torch.from_numpy(hp.from_device_order_host(got.cpu().numpy(), N, layout)))[0]
        hp.check_grad(name, got.numpy(), w, True)


def test_both_launches_give_the_same_bits():
    # 70 heads share one launch of both kinds, 280 do not: the order of the workgroups and the kernel of dQ touch no sum
    c, d = 250, 100
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
