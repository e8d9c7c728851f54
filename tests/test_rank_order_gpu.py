"""Uneven launches of more workgroups than the chip holds at once, up to a dozen rounds: taken up by ranks over all
heads.  Every head has the same rows, so every head's result is the first one's, bit for bit, and that is the oracle's;
numbers of heads that are and are no multiple of 8, whole chunks of ranks and the rest behind them."""
import numpy as np
import pytest
import torch

from oracle import striped_attention as orc
from paper_2311_09431_amd import binding as sa
from paper_2311_09431_amd import inputs
from tests import helpers as hp
from tests import routes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,c,d", [(64, 1152, 64), (75, 900, 128), (58, 1280, 32), (38, 1792, 100), (75, 1024, 256)])
def test_every_head_is_the_first(H, c, d):
    tiles = (c + 127) // 128
    assert 512 < tiles * H <= 3072
    a = routes.args(c, d, H)
    assert routes.forward(a) == routes.backward(a) == "128 rows" and routes.queries_by_rank(a) and routes.keys_by_rank(a)
    one = inputs.qkv(1, 1, c, d, c, torch.bfloat16, with_dout=True)
    q, k, v, g = (x.cuda().expand(1, H, c, d).contiguous() for x in one)
    o, lse = torch.empty(1, H, c, d, device="cuda"), torch.empty(1, H, c, device="cuda")
    shape = sa.shard_shape(q, c, lse)
    sa.sa_state_init(o, lse, shape)
    sa.sa_attn_step_fwd(q, k, v, o, lse, 0, 0, 1, sa.STRIPED, shape)
    delta, grads = torch.empty_like(lse), [torch.zeros_like(o) for _ in range(3)]
    sa.sa_bwd_preprocess(o, g, delta, shape)
    sa.sa_attn_step_bwd(q, k, v, g, lse, delta, *grads, 0, 0, 1, sa.STRIPED, shape)
    for x in (o, lse, *grads):
        assert torch.equal(x, x[:, :1].expand_as(x))
    q, k, v, g = (inputs.to_f64(x) for x in one)
    scale = 1.0 / np.sqrt(d)
    Ow, Lw = orc.causal_attention_bh(q, k, v, scale)
    assert hp.max_abs_err(o[:, :1].cpu().numpy(), Ow) <= 2e-2 and hp.max_abs_err(lse[:, :1].cpu().numpy(), Lw) <= 1e-3
    for name, got, w in zip(("dQ", "dK", "dV"), grads, orc.causal_attention_grad_bh(q, k, v, g, scale)):
        hp.check_grad(name, got[:, :1].cpu().numpy(), w, True)
