"""The library's own rules that choose a kernel, asked on the host (they launch nothing): tests say with
them which kernel a case reaches, so that a case meant for one cannot drift to another unnoticed."""
import ctypes

from paper_2311_09431_amd import binding as sa


class StepArgs(ctypes.Structure):          # csrc/sa_internal.h
    _fields_ = ([(n, ctypes.c_void_p) for n in ("q", "k", "v", "dout", "o", "lse", "delta", "dq", "dk", "dv")]
                + [(n, ctypes.c_int) for n in ("B", "H", "c", "d")]
                + [(n, ctypes.c_int64) for n in ("stride_b", "stride_h", "stat_stride_b", "stat_stride_h", "stride_s")]
                + [("H_kv", ctypes.c_int)]
                + [(n, ctypes.c_int64) for n in ("kv_stride_b", "kv_stride_h", "kv_stride_s")]
                + [("scale", ctypes.c_float)]
                + [(n, ctypes.c_int) for n in ("layout", "q_dev", "n_q", "kv_dev", "n_kv")]
                + [("q_shard", ctypes.c_int64), ("kv_shard", ctypes.c_int64), ("fresh", ctypes.c_bool)]
                + [("skip_bq", ctypes.c_int), ("skip_bk", ctypes.c_int)]
                + [("q_pos", ctypes.c_void_p), ("pos_stride_b", ctypes.c_int64), ("rope_log2_base", ctypes.c_double)])


def args(c, d, H, Hkv=None, B=1, q_dev=1, kv_dev=0, layout=sa.STRIPED, stride_s=None, kv_stride_s=None, N=1):
    """One step (N = 1), or a whole ring of N devices in one launch."""
    ring = N > 1
    a = StepArgs(B=B, H=H, c=c, d=d, H_kv=Hkv or H, scale=1.0, layout=layout, n_q=N, n_kv=N, fresh=ring,
                 q_dev=0 if ring else q_dev, kv_dev=0 if ring else kv_dev)
    a.stride_s, a.kv_stride_s = stride_s or d, kv_stride_s or d
    return a


def _ask(name, a, *more):
    signature = {int: "i", bool: "b"}
    fn = getattr(sa.lib(), "_ZN2sa%d%sERKNS_8StepArgsE%s" % (len(name), name, "".join(signature[type(m)] for m in more)))
    fn.restype, fn.argtypes = ctypes.c_bool, [ctypes.c_void_p] + [ctypes.c_int] * len(more)
    return fn(ctypes.byref(a), *more)


def f32(a, backward):
    """fp32 storage, up to 128 columns: the kind of kernel."""
    fn = getattr(sa.lib(), "_ZN2sa9f32_routeERKNS_8StepArgsEb")
    fn.restype, fn.argtypes = ctypes.c_int, [ctypes.c_void_p, ctypes.c_int]
    return ("fp32 instruction", "split", "128 rows", "128 rows, one wavefront")[fn(ctypes.byref(a), backward)]


def forward(a, dtype=sa.BF16):
    if not _ask("fwd_mfma_supported", a, dtype):
        return "short" if _ask("short_exact_wanted", a, dtype, False) else "fp32"
    return "split" if _ask("fwd_split_wanted", a) else "128 rows"


def backward(a, dtype=sa.BF16):
    if not _ask("bwd_mfma_supported", a, dtype):
        return "short" if _ask("short_exact_wanted", a, dtype, True) else "fp32"
    return "split" if _ask("bwd_split_wanted", a) else "128 rows"


def one_launch(a):
    """Whether both kinds of workgroups of a bf16 backward in 128-row tiles share a launch."""
    return _ask("bwd_one_launch", a)


def keys_by_rank(a):
    """The key-owning workgroups of a bf16 backward in 128-row tiles, by ranks over all heads."""
    return _ask("dkdv_by_rank", a)


def queries_by_rank(a):
    """The workgroups of a bf16 forward in 128-row tiles, by ranks over all heads."""
    return _ask("fwd_by_rank", a)
