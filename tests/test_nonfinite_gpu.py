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
from tests import routes

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
    (96, 96, 40, 64, BF16),         # ... more workgroups than compute units
    (256, 256, 33, 32, BF16),
    (400, 400, 40, 32, BF16),       # many heads up to 32 columns: a single forward block by the fp32 instruction
    (1, 1, 132, 132, BF16),         # above 128 columns, not whole 16-byte chunks
]
BLOCKS = [(1, 0, sa.STRIPED), (0, 1, sa.STRIPED), (1, 0, sa.CONTIGUOUS)]
INF, NAN = float("inf"), float("nan")


def close(name, got, want, tol=2e-5):
    for what in (np.isnan, np.isposinf, np.isneginf):
        assert np.array_equal(what(got), what(want)), (name, what.__name__, np.argwhere(what(got) != what(want))[:4])
    ok = np.isfinite(want)
    err = np.abs(got[ok] - want[ok]) / np.maximum(1.0, np.abs(want[ok]))
    assert err.size == 0 or err.max() <= tol, (name, float(err.max()))


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


def rows_backward(q, K, V, g, scale, lse, delta, n_keys):
    """Gradients of the pairs (a, b < n_keys[a])."""
    dq, dk, dv = np.zeros_like(q), np.zeros_like(K), np.zeros_like(V)
    for a, n in enumerate(n_keys):
        p = np.exp(scale * (K[:n] * q[a]).sum(1) - lse[a])
        ds = p * ((V[:n] * g[a]).sum(1) - delta[a])
        dq[a] = scale * (ds[:, None] * K[:n]).sum(0)
        dk[:n] += scale * ds[:, None] * q[a]
        dv[:n] += p[:, None] * g[a]
    return dq, dk, dv


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


def masked(t, at):
    """Elements of a later token that earlier rows of the same sub-tile must not see."""
    return {
        "v nan": lambda x: x["v"][:, :, at, 3].fill_(NAN),
        "v inf": lambda x: x["v"][:, :, at, 3].fill_(INF),
        "last v nan": lambda x: x["v"][:, :, -1, 0].fill_(NAN),
    }


def backward_kinds(t, at):
    first = t["q"][..., 0].abs() + 0.25
    return {
        "q nan": lambda x: x["q"][:, :, at, 2].fill_(NAN),
        "k nan": lambda x: x["k"][:, :, at, 1].fill_(NAN),
        "v inf": lambda x: x["v"][:, :, at, 3].fill_(INF),
        "k -inf": lambda x: (x["q"][..., 0].copy_(first), x["k"][:, :, at, 0].fill_(-INF)),
        "dO nan": lambda x: x["g"][:, :, at, 3].fill_(NAN),
        "dO -inf": lambda x: x["g"][:, :, at, 3].fill_(-INF),
        "delta nan": lambda x: x["delta"][:, :, at].fill_(NAN),
        "lse -inf": lambda x: x["lse"][:, :, at].fill_(-INF),
        "lse +inf": lambda x: x["lse"][:, :, at].fill_(INF),
        "first dO, last v": lambda x: (x["g"][:, :, 0, 0].fill_(INF), x["v"][:, :, -1, 1].fill_(NAN)),
    }


def large(t, at):
    """Finite, but beyond the largest bf16 number (fp32 storage)."""
    half = torch.full_like(t["q"][..., 0], 0.5)
    return {
        "k large": lambda x: (x["q"][..., 0].copy_(half), x["k"][:, :, at, 0].fill_(3.4e38)),
        "k large, negative": lambda x: (x["q"][..., 0].copy_(half), x["k"][:, :, at, 0].fill_(-3.4e38)),
        "v large": lambda x: x["v"][:, :, at, 3].fill_(3.4e38),
    }


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


def check_forward_step(route, block, kinds, tol=2e-5):
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
                close((name, fresh, "O"), o[0, h].cpu().numpy(), np.stack([w[0] for w in want]), tol)
                close((name, fresh, "LSE"), lse[0, h].cpu().numpy(), np.array([w[1] for w in want]), tol)


def check_backward_step(route, block, kinds):
    (H, Hkv, c, d, dtype), (q_dev, kv_dev, layout) = route, block
    t, at, scale, group = draw(H, Hkv, c, d, dtype), min(20, c - 2), 1.0 / np.sqrt(d), H // Hkv
    n_keys = [c if layout == sa.CONTIGUOUS else a + 1 - (kv_dev > q_dev) for a in range(c)]
    for name, poison in kinds(t, at).items():
        x = poisoned(t, poison)
        gq, gk, gv, gg, lse, delta = (x[n].cuda() for n in ("q", "k", "v", "g", "lse", "delta"))
        grads = [torch.zeros(y.shape, dtype=F32, device="cuda") for y in (gq, gk, gv)]
        shape = sa.shard_shape(gq, c, lse, kv=gk if Hkv != H else None)
        sa.sa_attn_step_bwd(gq, gk, gv, gg, lse, delta, *grads, q_dev, kv_dev, 2, layout, shape)
        torch.cuda.synchronize()
        for kvh in {0, Hkv - 1}:
            k, v = (inputs.to_f64(x[n][0, kvh]) for n in ("k", "v"))
            dk, dv = np.zeros((c, d)), np.zeros((c, d))
            for h in range(kvh * group, (kvh + 1) * group):
                q, g, l, de = (inputs.to_f64(x[n][0, h]) for n in ("q", "g", "lse", "delta"))
                dq, a, b = rows_backward(q, k, v, g, scale, l, de, n_keys)
                dk, dv = dk + a, dv + b
                close((name, "dQ"), grads[0][0, h].cpu().numpy(), dq)
            close((name, "dK"), grads[1][0, kvh].cpu().numpy(), dk)
            close((name, "dV"), grads[2][0, kvh].cpu().numpy(), dv)


def check_ring(route, layout, N, kinds, backward, tol=2e-5):
    """The drivers on the whole ring: every row over all shards."""
    H, Hkv, c, d, dtype = route
    S, scale, group = N * c, 1.0 / np.sqrt(d), H // Hkv
    t, at = draw(H, Hkv, S, d, dtype), S // 2 + 5
    for name, poison in kinds(t, at).items():
        x = poisoned(t, poison)
        p = {n: hp.to_device_order(x[n].cuda(), N, layout) for n in ("q", "k", "v", "g")}
        f32 = dict(dtype=F32, device="cuda")
        O, LSE, delta = torch.empty(1, H, S, d, **f32), torch.empty(1, H, S, **f32), torch.empty(1, H, S, **f32)
        shape = sa.shard_shape(p["q"], c, LSE, kv=p["k"] if Hkv != H else None)
        host = lambda y, h: hp.from_device_order_host(y[:, h:h + 1].cpu().numpy(), N, layout)[0, 0]
        sa.sa_ring_fwd(p["q"], p["k"], p["v"], O, LSE, N, layout, shape)
        if backward:        # with the statistics of the clean tensors
            y = {n: hp.to_device_order(t[n].cuda(), N, layout) for n in ("q", "k", "v")}
            sa.sa_ring_fwd(y["q"], y["k"], y["v"], O, LSE, N, layout, shape)
            grads = [torch.empty(z.shape, **f32) for z in (p["q"], p["k"], p["v"])]
            sa.sa_ring_bwd(p["q"], p["k"], p["v"], p["g"], O, LSE, delta, *grads, N, layout, shape)
        torch.cuda.synchronize()
        for kvh in {0, Hkv - 1}:
            k, v = (inputs.to_f64(x[n][0, kvh]) for n in ("k", "v"))
            dk, dv = np.zeros((S, d)), np.zeros((S, d))
            for h in range(kvh * group, (kvh + 1) * group):
                q, g = (inputs.to_f64(x[n][0, h]) for n in ("q", "g"))
                if not backward:
                    want = [row_forward(q[a], k[:a + 1], v[:a + 1], scale, np.zeros(d), -INF) for a in range(S)]
                    close((name, "O"), host(O, h), np.stack([w[0] for w in want]), tol)
                    close((name, "LSE"), host(LSE, h), np.array([w[1] for w in want]), tol)
                    continue
                dq, a, b = rows_backward(q, k, v, g, scale, host(LSE, h).astype(float), host(delta, h).astype(float),
                                         range(1, S + 1))
                dk, dv = dk + a, dv + b
                close((name, "dQ"), host(grads[0], h), dq)
            if backward:
                close((name, "dK"), host(grads[1], kvh), dk)
                close((name, "dV"), host(grads[2], kvh), dv)


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
    check_ring(route, layout, 2, swallowed, False)


@np_quiet
@pytest.mark.parametrize("block", BLOCKS)
@pytest.mark.parametrize("route", ROUTES)
def test_masked_values_stay_out_of_the_forward(route, block):
    check_forward_step(route, block, masked)


@np_quiet
@pytest.mark.parametrize("block", BLOCKS)
@pytest.mark.parametrize("route", ROUTES)
def test_masked_values_stay_out_of_the_gradients(route, block):
    check_backward_step(route, block, backward_kinds)


@np_quiet
@pytest.mark.parametrize("layout", [sa.STRIPED, sa.CONTIGUOUS])
@pytest.mark.parametrize("route", ROUTES[:2] + ROUTES[4:5] + ROUTES[6:8])
def test_masked_values_in_a_ring(route, layout):
    check_ring(route, layout, 2, masked, False)
    check_ring(route, layout, 2, lambda t, at: {n: f for n, f in backward_kinds(t, at).items() if "l" != n[0] and "delta" not in n}, True)


@np_quiet
@pytest.mark.parametrize("block", BLOCKS)
@pytest.mark.parametrize("route", [r for r in ROUTES if r[4] is F32])
def test_numbers_beyond_the_largest_bf16(route, block):
    check_forward_step(route, block, large)


@np_quiet
@pytest.mark.parametrize("layout", [sa.STRIPED, sa.CONTIGUOUS])
@pytest.mark.parametrize("route", [(2, 1, 160, 64, BF16), (1, 1, 128, 128, BF16), (1, 1, 130, 136, BF16),
                                   (260, 130, 160, 64, BF16), (260, 260, 128, 128, BF16), (260, 260, 130, 100, BF16)])
def test_the_128_row_kernels_leave_no_number_in_the_lse_of_such_a_row(route, layout):
    # O of a row with a NaN or +inf score is NaN there too; its LSE would pass for that of a row without keys.
    # (Few heads up to 128 columns: the split kernel, but for a block of one tile and d 64.)
    H, Hkv, c, d, _ = route
    if H == 260:
        for N in (1, 2):
            assert routes.forward(routes.args(c, d, H, Hkv, N=N, layout=layout)) == "128 rows"
    kinds = lambda t, at: {n: f for n, f in swallowed(t, at).items() if "-inf" not in n}
    for N in (1, 2):
        check_ring(route, layout, N, kinds, False, 2e-2)
    for block in BLOCKS:
        check_forward_step(route, block, kinds, 2e-2)


@np_quiet
@pytest.mark.parametrize("layout", [sa.STRIPED, sa.CONTIGUOUS])
@pytest.mark.parametrize("name", ["q", "k", "v", "g"])
def test_both_column_halves_in_a_workgroup_as_side_by_side(layout, name):
    # above 128 columns, bf16: what a NaN reaches in dQ, dK and dV is the same whether a launch is large enough for the
    # workgroups that hold both column halves of dK and dV or each head is a launch of its own
    H, c, d = 260, 160, 144
    t, f32 = draw(H, H, c, d, BF16), dict(dtype=F32, device="cuda")
    t[name][0, :, 70, 130] = NAN
    x = {n: t[n].cuda() for n in ("q", "k", "v", "g", "lse", "delta")}
    x["lse"] += 4.0
    play = lambda y, out: sa.sa_attn_step_bwd(y["q"], y["k"], y["v"], y["g"], y["lse"], y["delta"], *out, 1, 0, 2, layout,     # noqa: E731
                                              sa.shard_shape(y["q"], c, y["lse"]))
    whole = [torch.zeros(1, H, c, d, **f32) for _ in range(3)]
    play(x, whole)
    for h in (0, 7, H - 1):
        single = [torch.zeros(1, 1, c, d, **f32) for _ in range(3)]
        play({n: y[:, h:h + 1] for n, y in x.items()}, single)
        torch.cuda.synchronize()
        for got, want in zip(whole, single):
            got = got[:, h:h + 1]
            nan = torch.isnan(want)
            assert bool(nan.any()) or name != "q" and name != "k"
            assert torch.equal(torch.isnan(got), nan)
            # (products of one head summed in another order, in fp32)
            ok = ~nan
            assert float((got[ok] - want[ok]).norm()) <= 1e-5 * float(want[ok].norm())
