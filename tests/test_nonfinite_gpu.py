"""Infinities and NaN through the kernels of fp32 precision (fp32 storage, bf16 blocks below 128 rows,
bf16 shapes that the bf16 kernels do not take): they reach the rows that see them, as they would in a
sum over the allowed pairs alone, and no others.  A row with a NaN or +inf score is NaN in O and LSE; a
key at -inf has no weight; a later token's value stays out of earlier rows.  The reference forms every
row from its allowed keys only, in fp64."""
import numpy as np
import pytest
import torch

from paper_2311_09431_amd import binding as sa
from paper_2311_09431_amd import inputs
from tests import helpers as hp

pytestmark = pytest.mark.gpu

F32, BF16 = torch.float32, torch.bfloat16
ROUTES = [
    # H, H_kv, c, d, dtype
    (2, 1, 48, 64, F32),            # streamed rows split over four wavefronts
    (1, 1, 100, 36, F32),
    (1, 1, 70, 132, F32),           # ... over two (above 128 columns)
    (256, 256, 33, 132, F32),       # 128 rows a workgroup
    (256, 128, 40, 32, F32),        # three bf16 terms, four wavefronts
    (520, 520, 40, 68, F32),        # ... eight
    (2, 1, 48, 64, BF16),           # short bf16 blocks
    (1, 1, 100, 100, BF16),
    (96, 96, 40, 64, BF16),         # a single forward block of them by the fp32 instruction
    (256, 256, 33, 32, BF16),
    (1, 1, 132, 132, BF16),         # above 128 columns, not whole 16-byte chunks
]
BLOCKS = [(1, 0, sa.STRIPED), (0, 1, sa.STRIPED), (1, 0, sa.CONTIGUOUS)]
INF, NAN = float("inf"), float("nan")


def close(name, got, want):
    for what in (np.isnan, np.isposinf, np.isneginf):
        assert np.array_equal(what(got), what(want)), (name, what.__name__, np.argwhere(what(got) != what(want))[:4])
    ok = np.isfinite(want)
    err = np.abs(got[ok] - want[ok]) / np.maximum(1.0, np.abs(want[ok]))
    assert err.size == 0 or err.max() <= 2e-5, (name, float(err.max()))


def row_forward(q, K, V, scale, o0, lse0):
    """One query row over the keys it sees, folded into the state (o0, lse0)."""
    if len(K) == 0:
        return o0, lse0
    s = scale * (K * q).sum(1)
    m = float(np.maximum(lse0, np.max(s)))      # NaN if a score is
    if not np.isfinite(m):
        return np.full_like(o0, NAN), NAN       # NaN, +inf - (+inf), or every key at -inf and no state
    w0, w = np.exp(lse0 - m), np.exp(s - m)
    total = w0 + w.sum()
    old = w0 * o0 if w0 > 0 else 0.0
    return (old + (w[:, None] * V).sum(0)) / total, m + np.log(total)


def swallowed(t, at):
    """Scores that are no number, or minus infinity."""
    first = t["q"][..., 0].abs() + 0.25
    cases = {
        "q nan": lambda x: x["q"][:, :, at].fill_(NAN),
        "k nan": lambda x: x["k"][:, :, at, 1].fill_(NAN),
        "k +inf": lambda x: (x["q"][..., 0].copy_(first), x["k"][:, :, at, 0].fill_(INF)),
        "k -inf": lambda x: (x["q"][..., 0].copy_(first), x["k"][:, :, at, 0].fill_(-INF)),
        "all keys -inf": lambda x: (x["q"][..., 0].copy_(first), x["k"][..., 0].fill_(-INF)),
    }
    return cases


def draw(H, Hkv, rows, d, dtype):
    t = {n: inputs.gaussian((1, h, rows, d), 40 + i + rows + d, dtype)
         for i, (n, h) in enumerate((("q", H), ("k", Hkv), ("v", Hkv), ("g", H)))}
    t["lse"] = inputs.gaussian((1, H, rows), 50, F32) + 4.0
    t["delta"] = inputs.gaussian((1, H, rows), 51, F32)
    t["o"] = inputs.gaussian((1, H, rows, d), 52, F32)
    return t


def poisoned(t, poison):
    x = {n: y.clone() for n, y in t.items()}
    poison(x)
    return x


def check_forward_step(route, block, kinds):
    (H, Hkv, c, d, dtype), (q_dev, kv_dev, layout) = route, block
    t, at, scale = draw(H, Hkv, c, d, dtype), min(20, c - 2), 1.0 / np.sqrt(d)
    n_keys = [c if layout == sa.CONTIGUOUS else a + 1 - (kv_dev > q_dev) for a in range(c)]
    for name, poison in kinds(t, at).items():
        x = poisoned(t, poison)
        for fresh in (False, True):
            gq, gk, gv, o, lse = (x[n].cuda() for n in ("q", "k", "v", "o", "lse"))
            shape = sa.shard_shape(gq, c, lse, kv=gk if Hkv != H else None)
            if fresh:
                sa.sa_state_init(o, lse, shape)
            sa.sa_attn_step_fwd(gq, gk, gv, o, lse, q_dev, kv_dev, 2, layout, shape)
            torch.cuda.synchronize()
            for h in {0, H - 1}:
                q, k, v = (inputs.to_f64(x[n][0, i]) for n, i in (("q", h), ("k", h * Hkv // H), ("v", h * Hkv // H)))
                o0 = np.zeros((c, d)) if fresh else inputs.to_f64(x["o"][0, h])
                l0 = np.full(c, -INF) if fresh else inputs.to_f64(x["lse"][0, h])
                want = [row_forward(q[a], k[:n], v[:n], scale, o0[a], l0[a]) for a, n in enumerate(n_keys)]
                close((name, fresh, "O"), o[0, h].cpu().numpy(), np.stack([w[0] for w in want]))
                close((name, fresh, "LSE"), lse[0, h].cpu().numpy(), np.array([w[1] for w in want]))


def check_ring(route, layout, N, kinds):
    """The driver on the whole ring: every row over all shards."""
    H, Hkv, c, d, dtype = route
    S, scale = N * c, 1.0 / np.sqrt(d)
    t, at = draw(H, Hkv, S, d, dtype), c + 5
    for name, poison in kinds(t, at).items():
        x = poisoned(t, poison)
        p = {n: hp.to_device_order(x[n].cuda(), N, layout) for n in ("q", "k", "v")}
        f32 = dict(dtype=F32, device="cuda")
        O, LSE = torch.empty(1, H, S, d, **f32), torch.empty(1, H, S, **f32)
        shape = sa.shard_shape(p["q"], c, LSE, kv=p["k"] if Hkv != H else None)
        host = lambda y, h: hp.from_device_order_host(y[:, h:h + 1].cpu().numpy(), N, layout)[0, 0]
        sa.sa_ring_fwd(p["q"], p["k"], p["v"], O, LSE, N, layout, shape)
        torch.cuda.synchronize()
        for h in {0, H - 1}:
            q, k, v = (inputs.to_f64(x[n][0, i]) for n, i in (("q", h), ("k", h * Hkv // H), ("v", h * Hkv // H)))
            want = [row_forward(q[a], k[:a + 1], v[:a + 1], scale, np.zeros(d), -INF) for a in range(S)]
            close((name, "O"), host(O, h), np.stack([w[0] for w in want]))
            close((name, "LSE"), host(LSE, h), np.array([w[1] for w in want]))


np_quiet = pytest.mark.filterwarnings("ignore::RuntimeWarning")


@np_quiet
@pytest.mark.parametrize("block", BLOCKS)
@pytest.mark.parametrize("route", ROUTES)
def test_a_score_that_is_no_number_makes_its_rows_nan(route, block):
    check_forward_step(route, block, swallowed)


@np_quiet
@pytest.mark.parametrize("layout", [sa.STRIPED, sa.CONTIGUOUS])
@pytest.mark.parametrize("route", ROUTES)
def test_scores_that_are_no_numbers_in_a_ring(route, layout):
    check_ring(route, layout, 2, swallowed)
