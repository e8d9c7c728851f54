// C ABI of libstriped_attn: argument validation, mask classification, dispatch to
// the kernels, and the single-GPU ring drivers (Algorithm 1 played in sequence).
#include <math.h>

#include <algorithm>
#include <vector>

#include "sa_internal.h"

namespace {

using sa::StepArgs;

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

inline int64_t row_stride(const sa_shape* s) { return s->stride_s > 0 ? s->stride_s : s->d; }

// strides of one [B, heads, rows, d]-like tensor family
struct Geom { int heads; int64_t sb, sh, ss; };
inline Geom q_geom(const sa_shape* s) { return {s->H, s->stride_b, s->stride_h, row_stride(s)}; }
inline bool grouped(const sa_shape* s) { return s->H_kv > 0; }
inline Geom kv_geom(const sa_shape* s) {
    if (!grouped(s)) return q_geom(s);
    return {s->H_kv, s->kv_stride_b, s->kv_stride_h, s->kv_stride_s > 0 ? s->kv_stride_s : s->d};
}

// rows rows per (batch, head) must not overlap each other
int check_geom(const Geom& g, int B, int64_t rows, int d) {
    const int dmul = 4;      // rows are read four elements at a time (16 or 8 bytes)
    if (g.ss < d) return SA_ERR_SHAPE;
    // heads apart ([B, H, rows, d]-like) or interleaved within a row step ([B, rows, H, d]-like)
    const bool heads_apart = g.sh >= rows * g.ss;
    const bool heads_inside = g.sh >= d && g.ss >= (int64_t)g.heads * g.sh;
    if (!heads_apart && !heads_inside) return SA_ERR_SHAPE;
    if (B > 1 && g.sb < (heads_apart ? g.sh : rows * g.ss)) return SA_ERR_SHAPE;
    if (g.sb % dmul || g.sh % dmul || g.ss % dmul) return SA_ERR_ALIGN;
    return SA_OK;
}

int check_shape(const sa_shape* s) {
    if (!s) return SA_ERR_NULL;
    if (s->dtype != SA_F32 && s->dtype != SA_BF16) return SA_ERR_DTYPE;
    if (s->B < 1 || s->H < 1 || s->c < 1 || s->d < 1 || s->d > 256) return SA_ERR_SHAPE;
    if ((int64_t)s->B * s->H > 65535) return SA_ERR_SHAPE;
    if (s->d % 4) return SA_ERR_SHAPE;
    if (s->H_kv < 0 || (grouped(s) && s->H % s->H_kv)) return SA_ERR_SHAPE;
    if (s->stat_stride_h < s->c || (s->B > 1 && s->stat_stride_b < s->stat_stride_h)) return SA_ERR_SHAPE;
    if (int e = check_geom(q_geom(s), s->B, s->c, s->d)) return e;
    if (grouped(s))
        if (int e = check_geom(kv_geom(s), s->B, s->c, s->d)) return e;
    return SA_OK;
}

// the ring drivers address N shards of c rows inside the same tensors
int check_ring_extent(const sa_shape* s, int N) {
    const int64_t rows = (int64_t)N * s->c;
    if (s->stat_stride_h < rows) return SA_ERR_SHAPE;
    if (check_geom(q_geom(s), s->B, rows, s->d) || check_geom(kv_geom(s), s->B, rows, s->d))
        return SA_ERR_SHAPE;
    return SA_OK;
}

int check_step(int q_dev, int kv_dev, int N, int layout) {
    if (N < 1 || q_dev < 0 || q_dev >= N || kv_dev < 0 || kv_dev >= N) return SA_ERR_DEV;
    if (layout != SA_CONTIGUOUS && layout != SA_STRIPED) return SA_ERR_LAYOUT;
    return SA_OK;
}

// the block of query device q_dev and key device kv_dev
StepArgs make_args(const sa_shape* s, int q_dev = 0, int kv_dev = 0, int layout = SA_STRIPED) {
    StepArgs a{};
    a.layout = layout; a.q_dev = q_dev; a.n_q = 1; a.kv_dev = kv_dev; a.n_kv = 1;
    a.B = s->B; a.H = s->H; a.c = s->c; a.d = s->d;
    a.stride_b = s->stride_b; a.stride_h = s->stride_h;
    a.stat_stride_b = s->stat_stride_b; a.stat_stride_h = s->stat_stride_h;
    a.stride_s = row_stride(s);
    const Geom kv = kv_geom(s);
    a.H_kv = kv.heads; a.kv_stride_b = kv.sb; a.kv_stride_h = kv.sh; a.kv_stride_s = kv.ss;
    a.scale = s->softmax_scale > 0.f ? s->softmax_scale : 1.0f / sqrtf((float)s->d);
    return a;
}

int permute_common(const void* src, void* dst, int64_t outer, int64_t n_seq, int64_t inner_bytes,
                   int N, bool inverse, void* stream) {
    if (N < 1) return SA_ERR_DEV;
    if (outer < 0 || n_seq < 0 || inner_bytes < 1 || n_seq % N) return SA_ERR_SHAPE;
    if (outer == 0 || n_seq == 0) return SA_OK;   // empty: nothing to move, pointers may be NULL
    if (!src || !dst) return SA_ERR_NULL;
    if (src == dst) return SA_ERR_LAYOUT;
    int64_t al = 16;
    while (inner_bytes % al) al >>= 1;
    if ((reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst)) & (uintptr_t)(al - 1))
        return SA_ERR_ALIGN;
    return sa::launch_permute(src, dst, outer, n_seq, inner_bytes, N, inverse, (hipStream_t)stream) ==
                   hipSuccess ? SA_OK : SA_ERR_HIP;
}

// Emulated tile-skipping granularity (Sec. 3.1): both 0 (the kernels' own), or multiples of
// 128 dividing c on a shape the MFMA kernels take.
int check_skip(const sa_shape* s, int bq, int bk) {
    if (bq == 0 && bk == 0) return SA_OK;
    if (bq < 128 || bk < 128 || bq % 128 || bk % 128 || s->c % bq || s->c % bk) return SA_ERR_SHAPE;
    StepArgs a = make_args(s);
    return sa::fwd_mfma_supported(a, s->dtype) && sa::bwd_mfma_supported(a, s->dtype) ? SA_OK
                                                                                      : SA_ERR_SHAPE;
}

size_t elt_size(int dtype) { return dtype == SA_F32 ? 4 : 2; }

// HIP takes fewer than 2^32 threads a launch.  The kernels' grids are one-dimensional; at worst they
// hold one workgroup of 256 threads per 32 rows of each side (as many at d > 128, where a key-owning
// workgroup has 64 rows and half of the columns; the bf16 forward workgroups of 512 threads, on blocks of fewer
// than 128 rows or launches of a few workgroups, count as two; the fp32 ones of 512 threads per 32 rows are taken
// only where their launch fits: f32x3_split_supported).
constexpr int64_t kMostWorkgroups = (int64_t(1) << 24) - 1;
int64_t workgroups_per_kv_head(const StepArgs& a) {
    return ((int64_t)a.c / 32 + 2) * ((int64_t)a.n_q * (a.H / a.H_kv) * (a.c < 128 ? 2 : 1) + a.n_kv);
}
// Blocks of a launch that may hold more are played in parts of whole key/value heads and their groups.
template <typename Launch>
hipError_t in_parts(const StepArgs& a, int dtype, Launch launch) {
    const int64_t fit = std::max<int64_t>(1, kMostWorkgroups / workgroups_per_kv_head(a));
    if ((int64_t)a.B * a.H_kv <= fit) return launch(a);
    const int heads = (int)std::min<int64_t>(fit, a.H_kv), batches = (int)std::max<int64_t>(1, fit / a.H_kv);
    const int group = a.H / a.H_kv;
    const int64_t es = (int64_t)elt_size(dtype);
    for (int b = 0; b < a.B; b += batches)
        for (int h = 0; h < a.H_kv; h += heads) {
            StepArgs part = a;
            part.B = std::min(batches, a.B - b);
            part.H_kv = std::min(heads, a.H_kv - h);
            part.H = part.H_kv * group;
            const int64_t q = b * a.stride_b + (int64_t)h * group * a.stride_h, kv = b * a.kv_stride_b + h * a.kv_stride_h;
            const int64_t stat = b * a.stat_stride_b + (int64_t)h * group * a.stat_stride_h;
            auto in = [&](const void* p, int64_t at) -> const void* { return p ? (const char*)p + at * es : nullptr; };
            part.q = in(a.q, q); part.dout = in(a.dout, q); part.k = in(a.k, kv); part.v = in(a.v, kv);
            if (a.o) part.o = a.o + q;
            if (a.dq) part.dq = a.dq + q;
            if (a.dk) part.dk = a.dk + kv;
            if (a.dv) part.dv = a.dv + kv;
            part.lse = a.lse + stat;
            if (a.delta) part.delta = a.delta + stat;
            if (a.q_pos) part.q_pos = a.q_pos + b * a.pos_stride_b;
            if (hipError_t e = launch(part)) return e;
        }
    return hipSuccess;
}

hipError_t launch_fwd(const StepArgs& all, int dtype, hipStream_t st) {
    return in_parts(all, dtype, [&](const StepArgs& a) {
        if (!sa::fwd_mfma_supported(a, dtype)) return sa::launch_fwd_f32(a, dtype, st);
        return sa::fwd_split_wanted(a) ? sa::launch_fwd_split(a, st) : sa::launch_fwd_mfma(a, st);
    });
}
hipError_t launch_bwd(const StepArgs& all, int dtype, hipStream_t st) {
    return in_parts(all, dtype, [&](const StepArgs& a) {
        if (!sa::bwd_mfma_supported(a, dtype)) return sa::launch_bwd_f32(a, dtype, st);
        return sa::bwd_split_wanted(a) ? sa::launch_bwd_split(a, st) : sa::launch_bwd_mfma(a, st);
    });
}

int step_fwd(const void* q, const void* k, const void* v, float* o, float* lse, int q_dev, int kv_dev,
             int layout, const sa_shape* s, int bq, int bk, hipStream_t st, const int32_t* q_pos = nullptr,
             int64_t pos_stride_b = 0, float rope_base = 0.f) {
    StepArgs a = make_args(s, q_dev, kv_dev, layout);
    a.q = q; a.k = k; a.v = v; a.o = o; a.lse = lse;
    a.skip_bq = bq; a.skip_bk = bk;
    if (q_pos) {
        if (!sa::fwd_mfma_rope_supported(a, s->dtype)) return SA_ERR_SHAPE;
        a.q_pos = q_pos; a.pos_stride_b = pos_stride_b; a.rope_log2_base = log2((double)rope_base);
    }
    if (sa::block_kind(q_dev, kv_dev, layout) == sa::MASK_EMPTY) return SA_OK;   // nothing to launch
    return launch_fwd(a, s->dtype, st) == hipSuccess ? SA_OK : SA_ERR_HIP;
}

int step_bwd(const void* q, const void* k, const void* v, const void* dout, const float* lse,
             const float* delta, float* dq, float* dk, float* dv, int q_dev, int kv_dev, int layout,
             const sa_shape* s, int bq, int bk, hipStream_t st) {
    StepArgs a = make_args(s, q_dev, kv_dev, layout);
    if (sa::block_kind(q_dev, kv_dev, layout) == sa::MASK_EMPTY) return SA_OK;
    a.skip_bq = bq; a.skip_bk = bk;
    a.q = q; a.k = k; a.v = v; a.dout = dout; a.lse = const_cast<float*>(lse); a.delta = delta;
    a.dq = dq; a.dk = dk; a.dv = dv;
    return launch_bwd(a, s->dtype, st) == hipSuccess ? SA_OK : SA_ERR_HIP;
}

// The ring drivers without per-step timings: one launch per kernel for all blocks of the played
// devices, where rows are numbered in 31 bits and a key/value head's blocks fit a launch.  Else,
// and when the caller wants each step's time, one launch per block and kernel.
bool one_launch(const StepArgs& a, int N) {
    return (int64_t)N * a.c < (int64_t(1) << 31) && workgroups_per_kv_head(a) <= kMostWorkgroups;
}

// Event bookkeeping for the drivers' optional per-step timings.
struct StepTimer {
    std::vector<hipEvent_t> ev;
    std::vector<int> slot;
    bool on;
    explicit StepTimer(bool enabled) : on(enabled) {}
    bool begin(hipStream_t st, int s) {
        if (!on) return true;
        hipEvent_t a, b;
        if (hipEventCreate(&a) != hipSuccess) return false;
        if (hipEventCreate(&b) != hipSuccess) { (void)hipEventDestroy(a); return false; }
        ev.push_back(a); ev.push_back(b); slot.push_back(s);
        return hipEventRecord(a, st) == hipSuccess;
    }
    bool end(hipStream_t st) { return !on || hipEventRecord(ev.back(), st) == hipSuccess; }
    bool collect(hipStream_t st, float* out) {
        if (!on) return true;
        bool ok = hipStreamSynchronize(st) == hipSuccess;
        for (size_t i = 0; i < slot.size(); ++i) {
            float ms = 0.f;
            if (ok && hipEventElapsedTime(&ms, ev[2 * i], ev[2 * i + 1]) == hipSuccess) out[slot[i]] = ms;
            else ok = false;
        }
        return ok;
    }
    ~StepTimer() { for (hipEvent_t e : ev) (void)hipEventDestroy(e); }
};

}  // namespace

extern "C" {

int sa_stripe_permute(const void* src, void* dst, int64_t outer, int64_t n_seq, int64_t inner_bytes,
                      int32_t N, void* stream) {
    return permute_common(src, dst, outer, n_seq, inner_bytes, N, false, stream);
}

int sa_unstripe_permute(const void* src, void* dst, int64_t outer, int64_t n_seq, int64_t inner_bytes,
                        int32_t N, void* stream) {
    return permute_common(src, dst, outer, n_seq, inner_bytes, N, true, stream);
}

int sa_state_init(float* o, float* lse, const sa_shape* shape, void* stream) {
    if (!o || !lse) return SA_ERR_NULL;
    if (int e = check_shape(shape)) return e;
    if (!aligned16(o)) return SA_ERR_ALIGN;
    return sa::launch_state_init(o, lse, *shape, (hipStream_t)stream) == hipSuccess ? SA_OK : SA_ERR_HIP;
}

int sa_rope(const void* x, void* y, const int32_t* pos, int64_t pos_stride_b, const sa_shape* shape,
            float base, int32_t inverse, void* stream) {
    if (!x || !y || !pos) return SA_ERR_NULL;
    if (int e = check_shape(shape)) return e;
    if (pos_stride_b < 0 || (pos_stride_b > 0 && pos_stride_b < shape->c) || !(base > 1.f)) return SA_ERR_SHAPE;
    if (!aligned16(x) || !aligned16(y) || (reinterpret_cast<uintptr_t>(pos) & 3u)) return SA_ERR_ALIGN;
    return sa::launch_rope(x, y, pos, pos_stride_b, *shape, base, inverse != 0, (hipStream_t)stream) ==
                   hipSuccess ? SA_OK : SA_ERR_HIP;
}

int sa_attn_step_fwd_tiled(const void* q, const void* k, const void* v, float* o, float* lse,
                           int32_t q_dev, int32_t kv_dev, int32_t N, int32_t layout, const sa_shape* shape,
                           int32_t skip_bq, int32_t skip_bk, void* stream) {
    if (!q || !k || !v || !o || !lse) return SA_ERR_NULL;
    if (int e = check_shape(shape)) return e;
    if (int e = check_step(q_dev, kv_dev, N, layout)) return e;
    if (int e = check_skip(shape, skip_bq, skip_bk)) return e;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o)) return SA_ERR_ALIGN;
    return step_fwd(q, k, v, o, lse, q_dev, kv_dev, layout, shape, skip_bq, skip_bk, (hipStream_t)stream);
}

int sa_attn_step_fwd_rope(const void* q, const void* k, const void* v, float* o, float* lse,
                          const int32_t* q_pos, int64_t pos_stride_b, float rope_base, int32_t q_dev,
                          int32_t kv_dev, int32_t N, int32_t layout, const sa_shape* shape, void* stream) {
    if (!q || !k || !v || !o || !lse || !q_pos) return SA_ERR_NULL;
    if (int e = check_shape(shape)) return e;
    if (int e = check_step(q_dev, kv_dev, N, layout)) return e;
    if (pos_stride_b < 0 || (pos_stride_b > 0 && pos_stride_b < shape->c) || !(rope_base > 1.f)) return SA_ERR_SHAPE;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o) ||
        (reinterpret_cast<uintptr_t>(q_pos) & 3u))
        return SA_ERR_ALIGN;
    return step_fwd(q, k, v, o, lse, q_dev, kv_dev, layout, shape, 0, 0, (hipStream_t)stream, q_pos,
                    pos_stride_b, rope_base);
}

int sa_attn_step_fwd(const void* q, const void* k, const void* v, float* o, float* lse, int32_t q_dev,
                     int32_t kv_dev, int32_t N, int32_t layout, const sa_shape* shape, void* stream) {
    return sa_attn_step_fwd_tiled(q, k, v, o, lse, q_dev, kv_dev, N, layout, shape, 0, 0, stream);
}

int sa_finalize(const float* o, void* out, const sa_shape* shape, void* stream) {
    if (!o || !out) return SA_ERR_NULL;
    if (int e = check_shape(shape)) return e;
    if (!aligned16(o) || !aligned16(out)) return SA_ERR_ALIGN;
    return sa::launch_finalize(o, out, *shape, (hipStream_t)stream) == hipSuccess ? SA_OK : SA_ERR_HIP;
}

int sa_bwd_preprocess(const float* o, const void* dout, float* delta, const sa_shape* shape,
                      void* stream) {
    if (!o || !dout || !delta) return SA_ERR_NULL;
    if (int e = check_shape(shape)) return e;
    if (!aligned16(o) || !aligned16(dout)) return SA_ERR_ALIGN;
    return sa::launch_bwd_preprocess(o, dout, delta, *shape, shape->c, (hipStream_t)stream) == hipSuccess
               ? SA_OK : SA_ERR_HIP;
}

int sa_attn_step_bwd_tiled(const void* q, const void* k, const void* v, const void* dout,
                           const float* lse, const float* delta, float* dq, float* dk, float* dv,
                           int32_t q_dev, int32_t kv_dev, int32_t N, int32_t layout, const sa_shape* shape,
                           int32_t skip_bq, int32_t skip_bk, void* stream) {
    if (!q || !k || !v || !dout || !lse || !delta || !dq || !dk || !dv) return SA_ERR_NULL;
    if (int e = check_shape(shape)) return e;
    if (int e = check_step(q_dev, kv_dev, N, layout)) return e;
    if (int e = check_skip(shape, skip_bq, skip_bk)) return e;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(dout) || !aligned16(dq) ||
        !aligned16(dk) || !aligned16(dv))
        return SA_ERR_ALIGN;
    return step_bwd(q, k, v, dout, lse, delta, dq, dk, dv, q_dev, kv_dev, layout, shape, skip_bq, skip_bk,
                    (hipStream_t)stream);
}

int sa_attn_step_bwd(const void* q, const void* k, const void* v, const void* dout, const float* lse,
                     const float* delta, float* dq, float* dk, float* dv, int32_t q_dev, int32_t kv_dev,
                     int32_t N, int32_t layout, const sa_shape* shape, void* stream) {
    return sa_attn_step_bwd_tiled(q, k, v, dout, lse, delta, dq, dk, dv, q_dev, kv_dev, N, layout, shape,
                                  0, 0, stream);
}

int sa_ring_fwd_tiled(const void* Q, const void* K, const void* V, float* O, float* LSE, int32_t N,
                      int32_t layout, const sa_shape* shape, int32_t skip_bq, int32_t skip_bk,
                      int32_t q_dev_only, float* step_ms, void* stream) {
    if (!Q || !K || !V || !O || !LSE) return SA_ERR_NULL;
    if (int e = check_shape(shape)) return e;
    if (int e = check_skip(shape, skip_bq, skip_bk)) return e;
    if (N < 1 || q_dev_only >= N) return SA_ERR_DEV;
    if (layout != SA_CONTIGUOUS && layout != SA_STRIPED) return SA_ERR_LAYOUT;
    if (int e = check_ring_extent(shape, N)) return e;
    if (!aligned16(Q) || !aligned16(K) || !aligned16(V) || !aligned16(O)) return SA_ERR_ALIGN;
    hipStream_t st = (hipStream_t)stream;
    const size_t es = elt_size(shape->dtype);
    const int64_t shard = (int64_t)shape->c * row_stride(shape);     // elements between shards
    const int64_t kv_shard = (int64_t)shape->c * kv_geom(shape).ss;  // ... of K and V
    auto in_at = [&](const void* p, int dev) { return (const char*)p + (size_t)dev * shard * es; };
    auto kv_at = [&](const void* p, int dev) { return (const char*)p + (size_t)dev * kv_shard * es; };
    if (step_ms) for (int i = 0; i < N * N; ++i) step_ms[i] = 0.f;
    const int j0 = q_dev_only >= 0 ? q_dev_only : 0, j1 = q_dev_only >= 0 ? q_dev_only + 1 : N;
    StepArgs all = make_args(shape, j0, 0, layout);
    all.n_q = j1 - j0; all.n_kv = N; all.q_shard = shard; all.kv_shard = kv_shard; all.fresh = true;
    if (!step_ms && one_launch(all, N)) {
        all.q = in_at(Q, j0); all.k = K; all.v = V;
        all.o = O + j0 * shard; all.lse = LSE + (int64_t)j0 * shape->c;
        all.skip_bq = skip_bq; all.skip_bk = skip_bk;
        return launch_fwd(all, shape->dtype, st) == hipSuccess ? SA_OK : SA_ERR_HIP;
    }
    for (int j = j0; j < j1; ++j)
        if (sa::launch_state_init(O + j * shard, LSE + (int64_t)j * shape->c, *shape, st) != hipSuccess)
            return SA_ERR_HIP;
    StepTimer timer(step_ms != nullptr);
    for (int i = 0; i < N; ++i) {
        for (int j = j0; j < j1; ++j) {
            const int k = ((j - i) % N + N) % N;            // Algorithm 1: block held in round i
            if (!timer.begin(st, i * N + j)) return SA_ERR_HIP;
            int e = step_fwd(in_at(Q, j), kv_at(K, k), kv_at(V, k), O + j * shard,
                             LSE + (int64_t)j * shape->c, j, k, layout, shape, skip_bq, skip_bk, st);
            if (e) return e;
            if (!timer.end(st)) return SA_ERR_HIP;
        }
    }
    return timer.collect(st, step_ms) ? SA_OK : SA_ERR_HIP;
}

int sa_ring_fwd(const void* Q, const void* K, const void* V, float* O, float* LSE, int32_t N,
                int32_t layout, const sa_shape* shape, int32_t q_dev_only, float* step_ms, void* stream) {
    return sa_ring_fwd_tiled(Q, K, V, O, LSE, N, layout, shape, 0, 0, q_dev_only, step_ms, stream);
}

int sa_ring_bwd_tiled(const void* Q, const void* K, const void* V, const void* dO, const float* O,
                      const float* LSE, float* delta, float* dQ, float* dK, float* dV, int32_t N,
                      int32_t layout, const sa_shape* shape, int32_t skip_bq, int32_t skip_bk,
                      int32_t q_dev_only, float* step_ms, void* stream) {
    if (!Q || !K || !V || !dO || !O || !LSE || !delta || !dQ || !dK || !dV) return SA_ERR_NULL;
    if (int e = check_shape(shape)) return e;
    if (int e = check_skip(shape, skip_bq, skip_bk)) return e;
    if (N < 1 || q_dev_only >= N) return SA_ERR_DEV;
    if (layout != SA_CONTIGUOUS && layout != SA_STRIPED) return SA_ERR_LAYOUT;
    if (int e = check_ring_extent(shape, N)) return e;
    if (!aligned16(Q) || !aligned16(K) || !aligned16(V) || !aligned16(dO) || !aligned16(O) ||
        !aligned16(dQ) || !aligned16(dK) || !aligned16(dV))
        return SA_ERR_ALIGN;
    hipStream_t st = (hipStream_t)stream;
    const size_t es = elt_size(shape->dtype);
    const int64_t shard = (int64_t)shape->c * row_stride(shape);     // elements between shards
    const Geom kvg = kv_geom(shape);
    const int64_t kv_shard = (int64_t)shape->c * kvg.ss;             // ... of K, V, dK, dV
    auto in_at = [&](const void* p, int dev) { return (const char*)p + (size_t)dev * shard * es; };
    auto kv_at = [&](const void* p, int dev) { return (const char*)p + (size_t)dev * kv_shard * es; };
    if (step_ms) for (int i = 0; i < N * N; ++i) step_ms[i] = 0.f;
    const int j0 = q_dev_only >= 0 ? q_dev_only : 0, j1 = q_dev_only >= 0 ? q_dev_only + 1 : N;
    sa_shape kv_shape = *shape;          // dK and dV as a tensor family of their own
    kv_shape.H = kvg.heads; kv_shape.stride_b = kvg.sb; kv_shape.stride_h = kvg.sh; kv_shape.stride_s = kvg.ss;
    // rows first .. first + n - 1 of the devices' shards, as one tensor
    auto zero = [&](float* p, int64_t shard_elts, const sa_shape& s, int first, int n) {
        return n <= 0 || sa::launch_zero_f32(p + first * shard_elts, s, (int64_t)n * shape->c, st) == hipSuccess;
    };
    StepArgs all = make_args(shape, j0, 0, layout);
    all.n_q = j1 - j0; all.q_shard = shard; all.kv_shard = kv_shard; all.fresh = true;
    // key shards that some played device sees; contiguous layout: none further on than the last
    all.n_kv = layout == SA_STRIPED ? N : j1;
    if (!step_ms && one_launch(all, N)) {
        all.q = in_at(Q, j0); all.k = K; all.v = V; all.dout = in_at(dO, j0);
        all.lse = const_cast<float*>(LSE) + (int64_t)j0 * shape->c;
        all.delta = delta + (int64_t)j0 * shape->c;
        all.dq = dQ + j0 * shard; all.dk = dK; all.dv = dV;
        all.skip_bq = skip_bq; all.skip_bk = skip_bk;
        // what the kernels do not write: other devices' dQ, dK / dV of shards no played device sees
        if (!zero(dQ, shard, *shape, 0, j0) || !zero(dQ, shard, *shape, j1, N - j1) ||
            !zero(dK, kv_shard, kv_shape, all.n_kv, N - all.n_kv) ||
            !zero(dV, kv_shard, kv_shape, all.n_kv, N - all.n_kv) ||
            sa::launch_bwd_preprocess(O + j0 * shard, in_at(dO, j0), delta + (int64_t)j0 * shape->c, *shape,
                                      (int64_t)(j1 - j0) * shape->c, st) != hipSuccess)
            return SA_ERR_HIP;
        return launch_bwd(all, shape->dtype, st) == hipSuccess ? SA_OK : SA_ERR_HIP;
    }
    if (!zero(dQ, shard, *shape, 0, N) || !zero(dK, kv_shard, kv_shape, 0, N) ||
        !zero(dV, kv_shard, kv_shape, 0, N))
        return SA_ERR_HIP;
    for (int j = j0; j < j1; ++j)
        if (sa::launch_bwd_preprocess(O + j * shard, in_at(dO, j), delta + (int64_t)j * shape->c, *shape,
                                      shape->c, st) != hipSuccess)
            return SA_ERR_HIP;
    StepTimer timer(step_ms != nullptr);
    for (int i = 0; i < N; ++i) {
        for (int j = j0; j < j1; ++j) {
            const int k = ((j - i) % N + N) % N;
            if (!timer.begin(st, i * N + j)) return SA_ERR_HIP;
            int e = step_bwd(in_at(Q, j), kv_at(K, k), kv_at(V, k), in_at(dO, j),
                             LSE + (int64_t)j * shape->c, delta + (int64_t)j * shape->c, dQ + j * shard,
                             dK + k * kv_shard, dV + k * kv_shard, j, k, layout, shape, skip_bq, skip_bk,
                             st);
            if (e) return e;
            if (!timer.end(st)) return SA_ERR_HIP;
        }
    }
    return timer.collect(st, step_ms) ? SA_OK : SA_ERR_HIP;
}

int sa_ring_bwd(const void* Q, const void* K, const void* V, const void* dO, const float* O,
                const float* LSE, float* delta, float* dQ, float* dK, float* dV, int32_t N, int32_t layout,
                const sa_shape* shape, int32_t q_dev_only, float* step_ms, void* stream) {
    return sa_ring_bwd_tiled(Q, K, V, dO, O, LSE, delta, dQ, dK, dV, N, layout, shape, 0, 0, q_dev_only,
                             step_ms, stream);
}

int sa_step_mask(int32_t q_dev, int32_t kv_dev, int32_t N, int32_t layout, int32_t* kind, int32_t* off) {
    if (!kind || !off) return SA_ERR_NULL;
    if (int e = check_step(q_dev, kv_dev, N, layout)) return e;
    *kind = sa::block_kind(q_dev, kv_dev, layout);
    *off = sa::block_off(q_dev, kv_dev, layout);
    return SA_OK;
}

int64_t sa_step_pairs(int32_t q_dev, int32_t kv_dev, int32_t N, int32_t layout, int64_t c) {
    if (check_step(q_dev, kv_dev, N, layout) || c < 0) return -1;
    const int kind = sa::block_kind(q_dev, kv_dev, layout), off = sa::block_off(q_dev, kv_dev, layout);
    if (kind == sa::MASK_EMPTY) return 0;
    if (kind == sa::MASK_FULL) return c * c;
    return off ? c * (c - 1) / 2 : c * (c + 1) / 2;
}

int sa_step_tiles(int32_t q_dev, int32_t kv_dev, int32_t N, int32_t layout, int64_t c, int64_t skip_bq,
                  int64_t skip_bk, int64_t* computed, int64_t* total) {
    if (!computed || !total) return SA_ERR_NULL;
    if (int e = check_step(q_dev, kv_dev, N, layout)) return e;
    if (c < 1 || skip_bq < 1 || skip_bk < 1 || c % skip_bq || c % skip_bk) return SA_ERR_SHAPE;
    const int kind = sa::block_kind(q_dev, kv_dev, layout), off = sa::block_off(q_dev, kv_dev, layout);
    const int64_t nq = c / skip_bq, nk = c / skip_bk;
    *total = nq * nk;
    if (kind == sa::MASK_EMPTY) { *computed = 0; return SA_OK; }
    if (kind == sa::MASK_FULL) { *computed = nq * nk; return SA_OK; }
    // tile (r, s) holds an allowed pair iff its first key s*bk <= its last query (r+1)*bq - 1 - off
    int64_t n = 0;
    for (int64_t r = 0; r < nq; ++r) {
        const int64_t last = (r + 1) * skip_bq - 1 - off;       // last key any query of the tile sees
        if (last >= 0) n += (last / skip_bk + 1 < nk) ? last / skip_bk + 1 : nk;
    }
    *computed = n;
    return SA_OK;
}

int sa_device_props(int32_t* compute_units, int32_t* clock_khz, int64_t* memory_bytes) {
    if (!compute_units || !clock_khz || !memory_bytes) return SA_ERR_NULL;
    int dev = 0;
    hipDeviceProp_t prop;
    if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess) return SA_ERR_HIP;
    *compute_units = prop.multiProcessorCount;
    *clock_khz = prop.clockRate;
    *memory_bytes = (int64_t)prop.totalGlobalMem;
    return SA_OK;
}

const char* sa_status_str(int status) {
    switch (status) {
        case SA_OK: return "ok";
        case SA_ERR_NULL: return "null pointer";
        case SA_ERR_SHAPE: return "bad shape";
        case SA_ERR_DEV: return "device index out of range";
        case SA_ERR_DTYPE: return "unsupported dtype";
        case SA_ERR_LAYOUT: return "bad layout";
        case SA_ERR_ALIGN: return "misaligned pointer or stride";
        case SA_ERR_HIP: return "HIP call failed";
        default: return "unknown status";
    }
}

}  // extern "C"
