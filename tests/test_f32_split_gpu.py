"""fp32 launches of few rows: workgroups of 32 rows whose wavefronts (eight up to 64 columns, four above) stream
their sub-tiles of 32 rows by themselves, operands as three bf16 terms.  Against fp64 over the allowed pairs at the
edges of the sub-tiles, of a round of the wavefronts (4 and 8 sub-tiles) and of the columns (32, 64, 128 computed, chunks
of four), single steps on a running state, with grouped heads, infinities and NaN; the bounds are the fp32
configuration's.  And magnitudes that three bf16 terms do not cover."""
import pytest
import torch

from paper_2311_09431_amd import binding as sa
from paper_2311_09431_amd import inputs
from tests import routes
from tests import test_nonfinite_gpu as nf

pytestmark = [pytest.mark.gpu, nf.np_quiet]

ROUTES = [
    # H, H_kv, c, d, dtype
    (1, 1, 65, 4, torch.float32),
    (2, 2, 96, 32, torch.float32),
    (2, 1, 33, 36, torch.float32),
    (1, 1, 129, 100, torch.float32),
    (1, 1, 257, 128, torch.float32),
    (3, 3, 160, 100, torch.float32),
    (2, 2, 257, 64, torch.float32),
    (4, 2, 289, 28, torch.float32),
]


def reached(route):
    H, Hkv, c, d, _ = route
    return all(routes.f32(routes.args(c, d, H, Hkv), back) == "split" for back in (False, True))


@pytest.mark.parametrize("block", nf.BLOCKS)
@pytest.mark.parametrize("route", ROUTES)
def test_steps(route, block):
    assert reached(route)
    clean = lambda t, at: {"clean": lambda x: None}
    nf.check_forward_step(route, block, clean)
    nf.check_backward_step(route, block, clean)


@pytest.mark.parametrize("route", [ROUTES[2], ROUTES[4], ROUTES[6]])
def test_infinities_and_nan(route):
    for block in nf.BLOCKS:
        nf.check_forward_step(route, block, lambda t, at: {**nf.swallowed(t, at), **nf.masked(t, at)})
        nf.check_backward_step(route, block, nf.backward_kinds)


def test_rows_out_of_reach_are_others():
    # 32-bit byte offsets: the walk's last requests name up to 32 rows behind the last sub-tile
    for c, d in ((64, 64), (1000, 128)):
        behind = (c + 31) // 32 * 32 + 31
        for side in ("stride_s", "kv_stride_s"):
            pitches = [4 * ((1 << 31) // 16 // behind * i // 1000) for i in range(900, 1101)]
            taken = [p for p in pitches if routes.f32(routes.args(c, d, 1, **{side: p}), False) == "split"]
            assert taken and all(behind * 4 * p + 4 * d + 4096 < 1 << 31 for p in taken)
            assert len(taken) < len(pitches)


SMALL = [
    # H, c, d, 32-row workgroups
    (2, 257, 64, True),
    (3, 160, 100, True),
    (4, 289, 28, True),
    (64, 512, 128, False),
]


@pytest.mark.parametrize("small", ["q", "k", "v", "g"])
@pytest.mark.parametrize("H,c,d,split", SMALL)
def test_small_magnitudes(H, c, d, split, small):
    # three bf16 terms hold fewer than 24 bits of a number below 2^-109.  One operand scaled by a power of two: every output's
    # error in the 2-norm as without (3.5e-7 here, the fp32 instruction's 5.0e-7), not more than 1e-6
    for back in (False, True):
        assert routes.f32(routes.args(c, d, H, q_dev=0), back) in (("split",) if split else ("128 rows", "128 rows, one wavefront"))
    see = torch.ones(c, c, dtype=torch.bool, device="cuda").tril()
    for exponent in (-100, -105, -109, -112, -116, -120):
        x = {n: inputs.gaussian((1, H, c, d), 30 + i, device="cuda") for i, n in enumerate("qkvg")}
        x[small] *= 2.0 ** exponent
        o, lse, delta = torch.zeros_like(x["q"]), torch.empty(1, H, c, device="cuda"), torch.empty(1, H, c, device="cuda")
        grads = [torch.zeros_like(o) for _ in range(3)]
        shape = sa.shard_shape(x["q"], c, lse)
        sa.sa_state_init(o, lse, shape)
        sa.sa_attn_step_fwd(x["q"], x["k"], x["v"], o, lse, 0, 0, 1, sa.STRIPED, shape)
        sa.sa_bwd_preprocess(o, x["g"], delta, shape)
        sa.sa_attn_step_bwd(x["q"], x["k"], x["v"], x["g"], lse, delta, *grads, 0, 0, 1, sa.STRIPED, shape)
        q, k, v, g = (x[n].double() for n in "qkvg")
        t = lambda y: y.transpose(-1, -2).contiguous()      # noqa: E731
        p = (q @ t(k) * d ** -0.5).masked_fill(~see, -float("inf")).softmax(-1)
        ds = p * (g @ t(v) - (g * (p @ v)).sum(-1, keepdim=True)) * d ** -0.5
        for name, got, want in (("O", o, p @ v), ("dQ", grads[0], ds @ k), ("dK", grads[1], t(ds) @ q), ("dV", grads[2], t(p) @ g)):
            error = float((got.double() - want).norm() / want.norm())
            assert error <= 1e-6, (name, exponent, error)


@pytest.mark.parametrize("H,c,d,split", [(8, 2048, 64, True), (64, 2048, 128, False)])
def test_peaked_scores_take_no_longer(H, c, d, split):
    # scores of standard deviation 300 leave single keys whose every probability is below 2^-105 beside others: they are not
    # rows too small for their terms (each done over by itself: 13 times the launch's time)
    assert routes.f32(routes.args(c, d, H, q_dev=0), True) == ("split" if split else "128 rows")
    times = []
    for spread in (1, 300):
        q, k, v, g = (inputs.gaussian((1, H, c, d), 30 + i, device="cuda") for i in range(4))
        q *= spread
        o, lse, delta = torch.empty_like(q), torch.empty(1, H, c, device="cuda"), torch.empty(1, H, c, device="cuda")
        grads = [torch.empty_like(q) for _ in range(3)]
        shape = sa.shard_shape(q, c, lse)
        sa.sa_ring_fwd(q, k, v, o, lse, 1, sa.STRIPED, shape)
        call = lambda: sa.sa_ring_bwd(q, k, v, g, o, lse, delta, *grads, 1, sa.STRIPED, shape)      # noqa: E731
        call()
        taken = []
        for _ in range(5):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            for _ in range(4):
                call()
            end.record()
            torch.cuda.synchronize()
            taken.append(start.elapsed_time(end))
        times.append(min(taken))
        faint = [int(((x.abs().amax(-1) < 2.0 ** -105) & (x != 0).any(-1)).sum()) for x in grads[1:]]
    assert all(faint) and times[1] <= 2 * times[0], (faint, times)
