"""GPU parity of the fp32 matrix-core kernels (fp32 storage, and the bf16 shapes the bf16 kernels
do not take) at the edges of their 32-row sub-tiles, 64- and 128-row tiles and column counts, on
both splits of the work: 128 rows per workgroup (many heads) and streamed rows split over the
wavefronts (few heads).  fp32 arithmetic throughout, so bf16 inputs are held to the fp32 bounds
on O (fp32) and the gradients as well."""
import numpy as np
import pytest
import torch

from oracle import striped_attention as orc
from paper_2311_09431_amd import binding as sa
from paper_2311_09431_amd import inputs
from tests import helpers as hp

pytestmark = pytest.mark.gpu

CASES = [
    # B, H, c, d, N, dtype
    (1, 1, 1, 4, 3, torch.float32),
    (1, 2, 31, 32, 2, torch.float32),
    (1, 1, 32, 36, 2, torch.float32),
    (1, 1, 33, 64, 3, torch.float32),
    (1, 2, 126, 68, 2, torch.bfloat16),
    (1, 1, 128, 128, 2, torch.float32),
    (1, 1, 130, 132, 2, torch.bfloat16),        # above 128 columns, not whole 16-byte chunks
    (1, 1, 161, 256, 2, torch.float32),
    (1, 1, 260, 100, 2, torch.float32),
    (4, 64, 33, 32, 2, torch.float32),          # 256 heads: 128 rows per workgroup
    (4, 64, 65, 64, 2, torch.bfloat16),
    (2, 128, 40, 128, 2, torch.float32),
    (2, 128, 36, 200, 2, torch.float32),
    (1, 128, 130, 64, 2, torch.float32),        # two row tiles per head
]


@pytest.mark.parametrize("layout", [sa.CONTIGUOUS, sa.STRIPED])
@pytest.mark.parametrize("B,H,c,d,N,dtype", CASES)
def test_edges(layout, B, H, c, d, N, dtype):
    S, scale = N * c, 1.0 / np.sqrt(d)
    Q, K, V, dO = inputs.qkv(B, H, S, d, 7 * c + d, dtype, with_dout=True)
    g = [x.cuda() for x in (Q, K, V, dO)]
    O, LSE = hp.ring_forward_gpu(*g[:3], N, layout)
    grads = hp.ring_backward_gpu(*g, N, layout)
    torch.cuda.synchronize()
    # every head on small cases, first, middle and last of the many-head ones
    heads = range(B * H) if B * H <= 4 else [0, B * H // 2 + 1, B * H - 1]
    pick = lambda x: np.stack([np.asarray(x).reshape(B * H, *x.shape[2:])[i] for i in heads])[None]
    q, k, v, go = (pick(inputs.to_f64(x)) for x in (Q, K, V, dO))
    Ow, Lw = orc.causal_attention_bh(q, k, v, scale)
    host = lambda t: pick(hp.from_device_order_host(t.cpu().numpy(), N, layout))
    assert hp.max_abs_err(host(O), Ow) <= 1e-5
    assert hp.max_abs_err(host(LSE), Lw) <= 1e-5
    for name, got, want in zip(("dQ", "dK", "dV"), grads, orc.causal_attention_grad_bh(q, k, v, go, scale)):
        hp.check_grad(name, host(got), want, False)
