"""Head dimensions up to 32 in whole 16-byte chunks (32 columns computed): two k-steps and one column block in every
bf16 kernel.  Against the oracle at the edges of the 128-row and 32-row workgroups, of a chunk and of the columns, by
the split, the 128-row and the short-block kernels (few heads, many, blocks below 128 rows)."""
import numpy as np
import pytest
import torch

from paper_2311_09431_amd import binding as sa
from paper_2311_09431_amd import inputs
from tests import helpers as hp
from tests import routes

pytestmark = pytest.mark.gpu

CASES = [
    # H, c, d, N, forward steps, backward steps
    (2, 128, 32, 2, "128 rows", "split"),
    (1, 161, 24, 3, "split", "split"),
    (1, 1025, 32, 1, "split", "split"),
    (130, 129, 32, 2, "128 rows", "128 rows"),
    (96, 385, 8, 2, "128 rows", "128 rows"),
    (2, 97, 32, 2, "short", "short"),
]


@pytest.mark.parametrize("layout", [sa.CONTIGUOUS, sa.STRIPED])
@pytest.mark.parametrize("H,c,d,N,fwd,bwd", CASES)
def test_steps(layout, H, c, d, N, fwd, bwd):
    a = routes.args(c, d, H, layout=layout)
    assert (routes.forward(a), routes.backward(a)) == (fwd, bwd)
    scale = 1.0 / np.sqrt(d)
    Q, K, V, dO = inputs.qkv(1, H, N * c, d, c + d, torch.bfloat16, with_dout=True)
    g = [x.cuda() for x in (Q, K, V, dO)]
    O, LSE = hp.ring_forward_gpu(*g[:3], N, layout)
    steps, ring = (hp.ring_backward_gpu(*g, N, layout, use_driver=u) for u in (False, True))
    host = lambda t: hp.from_device_order_host(hp.some_heads(t)[0].cpu().numpy(), N, layout)
    q, k, v, go = hp.some_heads(Q, K, V, dO)
    Ow, Lw = hp.oracle_forward(q, k, v, scale)
    assert hp.max_abs_err(host(O), Ow) <= 2e-2 and hp.max_abs_err(host(LSE), Lw) <= 1e-3
    want = hp.oracle_backward(q, k, v, go, scale)
    for grads in (steps, ring):
        for name, got, w in zip(("dQ", "dK", "dV"), grads, want):
            hp.check_grad(name, host(got), w, True)
