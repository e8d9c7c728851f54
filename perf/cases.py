"""Timed cases of the Striped / Ring Attention ring step.

Three kinds of work, each through the public entry points as a user's program calls them:

  share    one sequence-parallel device's part of a ring, step by step: in a real ring the next
           K/V shard arrives from the neighbour between two steps, so the program owns the loop.
           State init, N forward steps, finalize; backward: delta, N backward steps that add to
           dQ and to the visiting shards' dK / dV.
  ring     the ring drivers on whole-sequence tensors (every device, or one of them), with the
           stripe permutation of the inputs in front when the layout is striped.
  permute  the stripe permutation and its inverse alone (activations, token and position ids).

Sizes are those of bench.py's workloads, of layer_bench.py's models and of the tests; inputs are
seeded standard Gaussians rounded once to the storage type, as everywhere in this repository.
"""
import math

import torch

from paper_2311_09431_amd import binding as sa
from paper_2311_09431_amd import inputs

LAYOUTS = {"striped": sa.STRIPED, "contiguous": sa.CONTIGUOUS}
DTYPES = {"bf16": torch.bfloat16, "fp32": torch.float32, "int32": torch.int32}

# kind, H_kv (0: as many as H), q_dev (-1: every device, ring only), order of the axes in memory,
# rope ("": none, "rows": q and k rotated by sa_rope, "fused": q rotated inside the forward step)
DEFAULTS = dict(kind="share", B=1, H=16, H_kv=0, d=128, c=4096, N=8, q_dev=7, dtype="bf16",
                layout="striped", order="bhsd", rope="", bwd=True)


def _case(name=None, **kw):
    case = dict(DEFAULTS, **kw)
    if name:
        case["name"] = name
    return case


def listed():
    return [
        # smallest: the fp32 configuration of 256 tokens on 4 devices, whole ring, where every
        # microsecond is a launch
        _case("tiny_fp32", kind="ring", H=1, d=64, c=64, N=4, q_dev=-1, dtype="fp32"),
        # bf16 shards shorter than one 128-row tile (short prompts split over 8 devices)
        _case("short_bf16", B=4, H=8, d=64, c=96, N=8, q_dev=3),
        # quick-check size: whole ring of 4096 tokens, forward and backward
        _case("ring_4k", kind="ring", H=2, c=1024, N=4, q_dev=-1),
        # 32k-token sequence on 8 devices, whole ring, forward (prefill)
        _case("ring_32k_fwd", kind="ring", H=16, c=4096, N=8, q_dev=-1, bwd=False),
        # fp32 training numerics at the shortest sequence length of the 1B model
        _case("ring_8k_fp32", kind="ring", H=16, c=2048, N=4, q_dev=-1, dtype="fp32"),
        # one device's share with 8 key/value heads for 32 query heads, 32k tokens
        _case("share_gqa_32k", H=32, H_kv=8, c=4096, N=8, q_dev=7),
        # 3B model (head dimension 100), rows as a projection writes them, rotary embedding,
        # one device's share through the drivers, 64k tokens
        _case("layer_3b_64k", kind="ring", H=32, d=100, c=8192, N=8, q_dev=7, order="bshd", rope="rows"),
        # ragged shards: 100000 tokens on 8 devices, head dimension 64
        _case("share_ragged_d64", H=16, d=64, c=12500, N=8, q_dev=5),
        # contiguous (Ring Attention) layout: full blocks, head dimension 256
        _case("share_contig_d256", H=8, d=256, c=8192, N=8, q_dev=7, layout="contiguous"),
        # longest sequence: 786k tokens on 16 devices, forward, rotation of q fused
        _case("share_786k_fwd", H=8, c=49152, N=16, q_dev=15, rope="fused", bwd=False),
        # largest: the default benchmark workload's 256k share, forward and backward
        _case("share_256k", H=32, c=32768, N=8, q_dev=7),
        # activations of a 256k sequence at head dimension 100 into device order and back
        _case("permute_256k_d100", kind="permute", H=32, d=100, c=32768, N=8),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["share", "share", "share", "ring", "ring", "permute"])
    if kind == "permute":
        case = _case(kind=kind, B=rng.choice([1, 1, 2]), H=rng.choice([1, 8, 16, 32]), N=rng.choice([2, 3, 4, 8, 16]),
                     d=rng.choice([1, 25, 64, 100, 128, 256]), dtype=rng.choice(["bf16", "bf16", "fp32", "int32"]),
                     layout="striped", bwd=False)
        case["c"] = max(1, _log_uniform(rng, 1024, 262144) // case["N"])
        while work(case)["bytes"] > work(listed()[-1])["bytes"]:
            case["c"] = case["c"] * 2 // 3
        return case
    fp32 = rng.random() < 0.2
    # 1 to 32 heads, shards from below one tile to the longest, every third of them a multiple of 128
    case = _case(kind=kind, B=rng.choice([1, 1, 2]), H=rng.choice([1, 2, 4, 8, 16, 32]),
                 d=rng.choice([32, 64, 128] if fp32 else [32, 64, 64, 100, 100, 128, 128, 128, 128, 256]),
                 c=_log_uniform(rng, 48, 2048 if fp32 else 49152), N=rng.choice([2, 3, 4, 8, 16]),
                 dtype="fp32" if fp32 else "bf16", layout=rng.choice(["striped", "striped", "contiguous"]),
                 order=rng.choice(["bhsd", "bshd"]), bwd=rng.random() < 0.6)
    if case["c"] > 128 and rng.random() < 0.5:
        case["c"] = case["c"] // 128 * 128
    case["q_dev"] = rng.randrange(case["N"]) if kind == "share" or rng.random() < 0.5 else -1
    if case["H"] > 2 and rng.random() < 0.25:
        case["H_kv"] = case["H"] // 4
    if rng.random() < 0.3:
        fused = kind == "share" and not fp32 and not case["bwd"] and case["d"] in (64, 128) and case["c"] % 128 == 0
        case["rope"] = "fused" if fused else "rows"
    # no more work than the largest listed case of the type; about 1 s of fp32 at most
    by_name = {x["name"]: x for x in listed()}
    most = work(by_name["ring_8k_fp32" if fp32 else "share_256k"])
    while work(case)["flops"] > most["flops"] or work(case)["bytes"] > most["bytes"]:
        case["c"] = max(1, case["c"] * 2 // 3)
        if case["rope"] == "fused":
            case["c"] = max(128, case["c"] // 128 * 128)
    return case


def _kv_heads(case):
    return case["H_kv"] or case["H"]


def _tensor(case, heads, rows, dtype, seed=None):
    """[B, heads, rows, d] tensor in the case's memory order: Gaussian (seed given) or empty."""
    seq_major = case["order"] == "bshd"
    shape = (case["B"], rows, heads, case["d"]) if seq_major else (case["B"], heads, rows, case["d"])
    x = (torch.empty(shape, dtype=dtype, device="cuda") if seed is None
         else inputs.gaussian(shape, seed, dtype, device="cuda"))
    return x.permute(0, 2, 1, 3) if seq_major else x


def _positions(case):
    """Position ids of the whole sequence in device order."""
    ids = torch.arange(case["N"] * case["c"], dtype=torch.int32, device="cuda")
    if case["layout"] == "striped":
        out = torch.empty_like(ids)
        sa.sa_stripe_permute(ids, out, case["N"], seq_axis=0)
        ids = out
    return ids


def prepare(case, seed):
    if case["kind"] == "permute":
        shape = (case["B"], case["H"], case["N"] * case["c"], case["d"])
        if case["dtype"] == "int32":
            g = torch.Generator(device="cuda")
            g.manual_seed(seed)
            x = torch.randint(0, 1 << 20, shape, generator=g, dtype=torch.int32, device="cuda")
        else:
            x = inputs.gaussian(shape, seed, DTYPES[case["dtype"]], device="cuda")
        return dict(case=case, x=x, y=torch.empty_like(x), z=torch.empty_like(x))

    H, Hkv, c, N, dev = case["H"], _kv_heads(case), case["c"], case["N"], case["q_dev"]
    dt, f32 = DTYPES[case["dtype"]], torch.float32
    rows = c if case["kind"] == "share" else N * c
    n_kv = N if case["kind"] == "share" else 1        # share: the visiting shards, each a tensor of its own
    s = dict(case=case, q=_tensor(case, H, rows, dt, 8 * seed))
    s["k"] = [_tensor(case, Hkv, rows, dt, 8 * (seed * 32 + i) + 1) for i in range(n_kv)]
    s["v"] = [_tensor(case, Hkv, rows, dt, 8 * (seed * 32 + i) + 2) for i in range(n_kv)]
    s["o"], s["out"] = _tensor(case, H, rows, f32), _tensor(case, H, rows, dt)
    s["lse"] = torch.empty(case["B"], H, rows, dtype=f32, device="cuda")
    if case["bwd"]:
        s["g"] = _tensor(case, H, rows, dt, 8 * seed + 3)
        s["delta"] = torch.empty_like(s["lse"])
        s["dq"] = _tensor(case, H, rows, f32)
        s["dk"], s["dv"] = ([_tensor(case, Hkv, rows, f32) for _ in range(n_kv)] for _ in range(2))
    kv = s["k"][0] if Hkv != H else None
    s["shape"] = sa.shard_shape(s["q"], c, s["lse"], kv=kv)
    if case["rope"]:
        pos = _positions(case)
        s["pos"] = pos[dev * c:(dev + 1) * c].contiguous() if dev >= 0 else pos
        # the projections' q and k, rotated by the pass ("fused": q only, in its step; the key
        # shards are in hand rotated)
        if case["rope"] == "rows":
            s["q_raw"], s["k_raw"] = (_tensor(case, n, rows, dt, 8 * seed + i) for n, i in ((H, 4), (Hkv, 5)))
        rope_rows = c if dev >= 0 else rows
        s["q_rope"] = sa.shard_shape(s["q"], rope_rows, s["lse"])
        s["k_rope"] = sa.shard_shape(s["k"][0], rope_rows)
        if case["bwd"]:
            s["dq_rope"], s["dk_rope"] = sa.shard_shape(s["dq"], rope_rows), sa.shard_shape(s["dk"][0], rope_rows)
            s["dq_in"], s["dk_in"] = torch.empty_like(s["dq"]), torch.empty_like(s["dk"][0])
    if case["kind"] == "ring":
        s["permute"] = case["layout"] == "striped" and case["order"] == "bhsd" and not case["rope"]
        names = ["q", "k", "v"] + (["g"] if case["bwd"] else [])
        s["ins"] = {n: s[n][0] if isinstance(s[n], list) else s[n] for n in names}
        s["ordered"] = {n: torch.empty_like(x) for n, x in s["ins"].items()} if s["permute"] else s["ins"]
    return s


def _run_share(s):
    case = s["case"]
    N, dev, layout, shape = case["N"], case["q_dev"], LAYOUTS[case["layout"]], s["shape"]
    q, ks, vs, o, lse = s["q"], s["k"], s["v"], s["o"], s["lse"]
    if case["rope"] == "rows":
        sa.sa_rope(s["q_raw"], q, s["pos"], s["q_rope"])
        sa.sa_rope(s["k_raw"], ks[dev], s["pos"], s["k_rope"])
    sa.sa_state_init(o, lse, shape)
    for i in range(N):
        k = (dev - i) % N
        if case["rope"] == "fused":
            sa.sa_attn_step_fwd_rope(q, ks[k], vs[k], o, lse, s["pos"], dev, k, N, layout, shape)
        else:
            sa.sa_attn_step_fwd(q, ks[k], vs[k], o, lse, dev, k, N, layout, shape)
    sa.sa_finalize(o, s["out"], shape)
    res = dict(o=o, lse=lse, out=s["out"])
    if case["bwd"]:
        sa.sa_bwd_preprocess(o, s["g"], s["delta"], shape)
        s["dq"].zero_()
        for i in range(N):
            k = (dev - i) % N
            s["dk"][k].zero_()          # the accumulators that travel with the visiting shard
            s["dv"][k].zero_()
            sa.sa_attn_step_bwd(q, ks[k], vs[k], s["g"], lse, s["delta"], s["dq"], s["dk"][k], s["dv"][k],
                                dev, k, N, layout, shape)
        res.update(dq=s["dq"], dk=s["dk"], dv=s["dv"])
        if case["rope"] == "rows":
            sa.sa_rope(s["dq"], s["dq_in"], s["pos"], s["dq_rope"], inverse=True)
            sa.sa_rope(s["dk"][dev], s["dk_in"], s["pos"], s["dk_rope"], inverse=True)
            res.update(dq_in=s["dq_in"], dk_in=s["dk_in"])
    return res


def _run_ring(s):
    case = s["case"]
    N, c, dev, layout, shape = case["N"], case["c"], case["q_dev"], LAYOUTS[case["layout"]], s["shape"]
    x = s["ordered"]
    if s["permute"]:
        for n, src in s["ins"].items():
            sa.sa_stripe_permute(src, x[n], N)
    q, k, v = x["q"], x["k"], x["v"]
    own = slice(dev * c, (dev + 1) * c) if dev >= 0 else slice(None)
    if case["rope"]:        # the played rows; other devices' key shards are in hand rotated
        sa.sa_rope(s["q_raw"][:, :, own], q[:, :, own], s["pos"], s["q_rope"])
        sa.sa_rope(s["k_raw"][:, :, own], k[:, :, own], s["pos"], s["k_rope"])
    sa.sa_ring_fwd(q, k, v, s["o"], s["lse"], N, layout, shape, dev)
    for j in range(N) if dev < 0 else [dev]:
        rows = slice(j * c, (j + 1) * c)
        sa.sa_finalize(s["o"][:, :, rows], s["out"][:, :, rows], shape)
    # one device's part fills its own rows only
    res = dict(o=s["o"][:, :, own], lse=s["lse"][:, :, own], out=s["out"][:, :, own])
    if case["bwd"]:
        sa.sa_ring_bwd(q, k, v, x["g"], s["o"], s["lse"], s["delta"], s["dq"], s["dk"][0], s["dv"][0], N, layout,
                       shape, dev)
        res.update(dq=s["dq"], dk=s["dk"][0], dv=s["dv"][0])
        if case["rope"]:
            sa.sa_rope(s["dq"][:, :, own], s["dq_in"][:, :, own], s["pos"], s["dq_rope"], inverse=True)
            sa.sa_rope(s["dk"][0][:, :, own], s["dk_in"][:, :, own], s["pos"], s["dk_rope"], inverse=True)
            res.update(dq_in=s["dq_in"][:, :, own], dk_in=s["dk_in"][:, :, own])
    return res


def run(state):
    kind = state["case"]["kind"]
    if kind == "permute":
        N = state["case"]["N"]
        sa.sa_stripe_permute(state["x"], state["y"], N)
        sa.sa_unstripe_permute(state["y"], state["z"], N)
        return dict(striped=state["y"], back=state["z"])
    return _run_share(state) if kind == "share" else _run_ring(state)


def _pairs(case):
    N, layout = case["N"], LAYOUTS[case["layout"]]
    devs = range(N) if case["q_dev"] < 0 else [case["q_dev"]]
    return sum(sa.sa_step_pairs(j, k, N, layout, case["c"]) for j in devs for k in range(N))


def work(case):
    B, H, Hkv, d, c, N = case["B"], case["H"], _kv_heads(case), case["d"], case["c"], case["N"]
    es = 2 if case["dtype"] == "bf16" else 4
    if case["kind"] == "permute":
        return {"bytes": 4 * B * H * N * c * d * es, "flops": 0}
    q_rows = B * H * d * c * (N if case["q_dev"] < 0 else 1)
    kv_rows = B * Hkv * d * c * N
    # q in, o and out, lse; k and v in; backward: dO in, dQ out, dK and dV out
    n_bytes = q_rows * (2 * es + 4) + q_rows // d * 4 + 2 * kv_rows * es
    if case["bwd"]:
        n_bytes += q_rows * (es + 4) + 2 * kv_rows * 4
    return {"bytes": n_bytes, "flops": _pairs(case) * B * H * d * (14 if case["bwd"] else 4)}


def tolerance(case):
    if case["kind"] == "permute":
        return "exact"
    # bf16: probabilities and dS are rounded to bf16 before their products (2^-9 of each term)
    return {"rel": 1e-2} if case["dtype"] == "bf16" else {"rel": 1e-5}
