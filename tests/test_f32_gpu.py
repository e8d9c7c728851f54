"""GPU parity of fp32 storage and of the bf16 shapes the bf16 kernels do not take, at the edges of 32-row
sub-tiles, 64- and 128-row tiles and column counts, few heads and many.  fp32 precision throughout, so
bf16 inputs are held to the fp32 bounds on O (fp32) and the gradients as well.  test_edges meets the fp32
matrix-core kernels with the streamed rows split over the wavefronts (few heads), with 128 rows per
workgroup (many heads above 128 columns), and where fp32 launches fill the chip the three-term kernels
(up to 128 columns); bf16 blocks below 128 rows are other kernels' in part (their own test), so
test_rows_far_apart meets the fp32 kernels' bf16 forms: rows too far apart for the bf16 kernels' 32-bit
tile addresses."""
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
    (4, 64, 33, 32, 2, torch.float32),          # 256 heads: three terms
    (4, 64, 65, 64, 2, torch.bfloat16),         # (short blocks on the bf16 matrix cores)
    (4, 128, 65, 32, 2, torch.bfloat16),        # ... 128 rows per workgroup (forward steps)
    (2, 128, 40, 128, 2, torch.float32),
    (2, 128, 36, 200, 2, torch.float32),        # ... 128 rows per workgroup
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


@pytest.mark.parametrize("H,c,d", [(1, 128, 32), (2, 130, 64), (1, 129, 128), (256, 128, 32), (256, 128, 64), (256, 128, 128)])
def test_rows_far_apart(H, c, d):
    # rows of K, V (and dK, dV) so far apart that 128 of them span 2^31 bytes: few heads, and 256 of them
    # side by side within a row (128 rows per workgroup)
    pitch = (1 << 31) // (2 * 128) + 64
    wide = lambda dtype: torch.empty(c * pitch, dtype=dtype, device="cuda").as_strided((1, H, c, d), (c * pitch, d, pitch, 1))
    q, g, k0, v0 = (inputs.gaussian((1, H, c, d), 80 + d + i, torch.bfloat16) for i in range(4))
    gq, gg, k, v, dk, dv = q.cuda(), g.cuda(), wide(q.dtype), wide(q.dtype), wide(torch.float32), wide(torch.float32)
    k.copy_(k0), v.copy_(v0), dk.zero_(), dv.zero_()
    f32 = dict(dtype=torch.float32, device="cuda")
    o, lse, delta, dq = (torch.empty(*s, **f32) for s in ((1, H, c, d), (1, H, c), (1, H, c), (1, H, c, d)))
    dq.zero_()
    shape = sa.shard_shape(gq, c, lse, kv=k)
    sa.sa_state_init(o, lse, shape)
    sa.sa_attn_step_fwd(gq, k, v, o, lse, 0, 0, 1, sa.CONTIGUOUS, shape)
    sa.sa_bwd_preprocess(o, gg, delta, shape)
    sa.sa_attn_step_bwd(gq, k, v, gg, lse, delta, dq, dk, dv, 0, 0, 1, sa.CONTIGUOUS, shape)
    torch.cuda.synchronize()
    heads = sorted({0, H // 2, H - 1})
    pick = lambda x: inputs.to_f64(x[:, heads].cpu())
    Ow, Lw = orc.causal_attention_bh(pick(q), pick(k0), pick(v0), 1.0 / np.sqrt(d))
    assert hp.max_abs_err(pick(o), Ow) <= 1e-5
    assert hp.max_abs_err(pick(lse), Lw) <= 1e-5
    for name, got, want in zip(("dQ", "dK", "dV"), (dq, dk, dv),
                               orc.causal_attention_grad_bh(pick(q), pick(k0), pick(v0), pick(g), 1.0 / np.sqrt(d))):
        hp.check_grad(name, pick(got), want, False)
