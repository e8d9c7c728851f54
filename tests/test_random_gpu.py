"""A seeded sweep over shapes the hand-picked cases may miss: random batch, heads, block size,
device count, head dimension, storage type, softmax scale and layout, forward and backward,
each against the fp64 oracle with the usual tolerances.  Half of the bf16 cases are built to
take the matrix-core kernels (here c a multiple of 128, d <= 128), the rest the generic ones."""
import numpy as np
import pytest
import torch

from paper_2311_09431_amd import binding as sa
from paper_2311_09431_amd import inputs
from tests import helpers as hp
from tests import routes

pytestmark = pytest.mark.gpu


def _cases(n, seed):
    rng = np.random.default_rng(seed)
    out = []
    for i in range(n):
        N = int(rng.choice([1, 2, 3, 4, 5, 8]))
        mfma = bool(i % 2)
        if mfma:
            c = 128 * int(rng.integers(1, 5))
            d = int(rng.choice([128, 128, 100, 64, 96, 32]))
            dtype = torch.bfloat16
        else:
            c = int(rng.integers(1, 90))
            d = 4 * int(rng.integers(1, 41))
            dtype = torch.float32 if rng.random() < 0.6 else torch.bfloat16
        B, H = int(rng.integers(1, 3)), int(rng.integers(1, 4))
        layout = sa.STRIPED if rng.random() < 0.6 else sa.CONTIGUOUS
        scale = None if rng.random() < 0.5 else float(rng.uniform(0.02, 0.3))
        out.append((B, H, c, N, d, dtype, layout, scale, int(rng.integers(1, 10 ** 6))))
    return out


@pytest.mark.parametrize("case", _cases(24, 2311_09431), ids=lambda c: "B%dH%dc%dN%dd%d" % c[:5])
def test_random_shapes_forward_and_backward(case):
    B, H, c, N, d, dtype, layout, scale, seed = case
    S = c * N
    Q, K, V, dO = inputs.qkv(B, H, S, d, seed, dtype, with_dout=True)
    sc = scale if scale else 1.0 / np.sqrt(d)
    Qg, Kg, Vg, Gg = (x.cuda() for x in (Q, K, V, dO))
    Qp, Kp, Vp, Gp = (hp.to_device_order(x, N, layout) for x in (Qg, Kg, Vg, Gg))
    O = torch.empty(B, H, S, d, dtype=torch.float32, device="cuda")
    LSE = torch.empty(B, H, S, dtype=torch.float32, device="cuda")
    delta = torch.empty_like(LSE)
    grads = [torch.empty_like(O) for _ in range(3)]
    shape = sa.shard_shape(Qp, c, LSE, scale)
    sa.sa_ring_fwd(Qp, Kp, Vp, O, LSE, N, layout, shape)
    sa.sa_ring_bwd(Qp, Kp, Vp, Gp, O, LSE, delta, *grads, N, layout, shape)
    torch.cuda.synchronize()
    Q, K, V, dO, O, LSE, *grads = hp.some_heads(Q, K, V, dO, O, LSE, *grads)
    back = lambda t: hp.from_device_order_host(t.cpu().numpy(), N, layout)
    bf16 = dtype == torch.bfloat16
    Ow, Lw = hp.oracle_forward(Q, K, V, sc)
    assert hp.max_abs_err(back(O), Ow) <= (2e-2 if bf16 else 1e-5)
    assert hp.max_abs_err(back(LSE), Lw) <= (1e-3 if bf16 else 1e-5)
    for g, w in zip(grads, hp.oracle_backward(Q, K, V, dO, sc)):
        hp.check_grad("gradient", back(g), w, bf16)


def _many_head_cases(n, seed):
    """Launches of more than 256 row tiles on both sides: none takes the split kernels."""
    rng = np.random.default_rng(seed)
    out = []
    while len(out) < n:
        N, c = int(rng.integers(1, 4)), int(rng.integers(128, 400))
        d = int(rng.choice([128, 100, 64, 96, 32, 120, 36, 256, 136]))
        if rng.random() < 0.4:
            c = c // 128 * 128
        while (c * d * 2) % 16:
            c += 1
        tiles = (c + 127) // 128 * N
        H = 256 // tiles + int(rng.integers(1, 8))
        layout = sa.STRIPED if rng.random() < 0.6 else sa.CONTIGUOUS
        out.append((1, H, c, N, d, torch.bfloat16, layout, None if rng.random() < 0.5 else float(rng.uniform(0.02, 0.3)),
                    int(rng.integers(1, 10 ** 6))))
    return out


@pytest.mark.parametrize("case", _many_head_cases(12, 94312), ids=lambda c: "B%dH%dc%dN%dd%d" % c[:5])
def test_random_shapes_of_many_heads(case):
    B, H, c, N, d, dtype, layout = case[:7]
    a = routes.args(c, d, H, N=N, layout=layout)
    assert routes.forward(a) == routes.backward(a) == "128 rows"
    test_random_shapes_forward_and_backward(case)


def _grouped_cases(n, seed):
    rng = np.random.default_rng(seed)
    out = []
    for i in range(n):
        N = int(rng.choice([1, 2, 3, 4]))
        if i % 2:
            c, d, dtype = 128 * int(rng.integers(1, 4)), int(rng.choice([128, 100, 64])), torch.bfloat16
        else:
            c, d = int(rng.integers(1, 70)), 4 * int(rng.integers(1, 33))
            dtype = torch.float32 if rng.random() < 0.5 else torch.bfloat16
        H_kv, group = int(rng.integers(1, 4)), int(rng.integers(1, 5))
        layout = sa.STRIPED if rng.random() < 0.6 else sa.CONTIGUOUS
        out.append((int(rng.integers(1, 3)), H_kv * group, H_kv, c, N, d, dtype, layout, bool(rng.random() < 0.5),
                    int(rng.integers(1, 10 ** 6))))
    return out


@pytest.mark.parametrize("case", _grouped_cases(12, 9431), ids=lambda c: "B%dH%dkv%dc%dN%dd%d" % c[:6])
def test_random_grouped_head_shapes(case):
    # fewer key/value heads than query heads, in [B, heads, S, d] or [B, S, heads, d] storage
    import oracle.striped_attention as orc
    B, H, H_kv, c, N, d, dtype, layout, seq_major, seed = case
    S = c * N
    Q = inputs.gaussian((B, H, S, d), seed, dtype)
    K = inputs.gaussian((B, H_kv, S, d), seed + 1, dtype)
    V = inputs.gaussian((B, H_kv, S, d), seed + 2, dtype)
    dO = inputs.gaussian((B, H, S, d), seed + 3, dtype)
    dev = [hp.to_device_order(x.cuda(), N, layout) for x in (Q, K, V, dO)]
    if seq_major:
        dev = [x.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3) for x in dev]
    Qp, Kp, Vp, Gp = dev
    O = torch.empty_like(Qp, dtype=torch.float32)
    LSE = torch.empty(B, H, S, dtype=torch.float32, device="cuda")
    delta = torch.empty_like(LSE)
    dQ = torch.empty_like(O)
    dK, dV = (torch.empty_like(Kp, dtype=torch.float32) for _ in range(2))
    shape = sa.shard_shape(Qp, c, LSE, None, kv=Kp)
    sa.sa_ring_fwd(Qp, Kp, Vp, O, LSE, N, layout, shape)
    sa.sa_ring_bwd(Qp, Kp, Vp, Gp, O, LSE, delta, dQ, dK, dV, N, layout, shape)
    torch.cuda.synchronize()
    back = lambda t: hp.from_device_order_host(t.cpu().numpy(), N, layout)
    bf16 = dtype == torch.bfloat16
    f = [inputs.to_f64(x) for x in (Q, K, V, dO)]
    sc = 1.0 / np.sqrt(d)
    Ow, Lw = orc.causal_attention_gqa(f[0], f[1], f[2], sc)
    assert hp.max_abs_err(back(O), Ow) <= (2e-2 if bf16 else 1e-5)
    assert hp.max_abs_err(back(LSE), Lw) <= (1e-3 if bf16 else 1e-5)
    for g, w in zip((dQ, dK, dV), orc.causal_attention_gqa_grad(*f, sc)):
        hp.check_grad("gradient", back(g), w, bf16)


def _mixed_cases(n, seed):
    """Everything at once: block sizes on, off and below the 128-row tiles, grouped heads, both
    memory orders (shard pointers kept 16-byte aligned, as the entry points require)."""
    rng = np.random.default_rng(seed)
    out = []
    for i in range(n):
        N = int(rng.choice([1, 2, 3, 4, 6]))
        kind = i % 3
        if kind == 0:
            c, d, dtype = 128 * int(rng.integers(1, 5)), int(rng.choice([128, 100, 64, 4, 120])), torch.bfloat16
        elif kind == 1:
            c, d, dtype = int(rng.integers(128, 600)), int(rng.choice([128, 100, 64, 32])), torch.bfloat16
        else:
            c, d = int(rng.integers(1, 128)), 4 * int(rng.integers(1, 65))
            dtype = torch.float32 if rng.random() < 0.5 else torch.bfloat16
        if c * N > 2200:
            N = max(1, 2200 // c)
        H_kv, group = int(rng.integers(1, 4)), int(rng.choice([1, 1, 2, 4]))
        seq_major = bool(rng.random() < 0.4)
        es = 2 if dtype == torch.bfloat16 else 4
        while (c * d * es) % 16 or (seq_major and (c * H_kv * d * es) % 16):
            c += 1
        layout = sa.STRIPED if rng.random() < 0.6 else sa.CONTIGUOUS
        out.append((int(rng.integers(1, 3)), H_kv * group, H_kv, c, N, d, dtype, layout, seq_major,
                    int(rng.integers(1, 10 ** 6))))
    return out


@pytest.mark.parametrize("case", _mixed_cases(18, 23110), ids=lambda c: "B%dH%dkv%dc%dN%dd%d" % c[:6])
def test_random_mixed_shapes(case):
    test_random_grouped_head_shapes(case)
