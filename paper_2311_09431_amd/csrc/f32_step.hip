// Ring-step kernels on the CDNA4 fp32 matrix cores (v_mfma_f32_32x32x2_f32: fp32 operands, fp32
// accumulation): any head dimension up to 256, any block size, fp32 or bf16 inputs.  They serve
// fp32 storage above 128 columns and launches of few rows below (error budget 1e-5, so no reduced-precision products and the accurate
// expf / logf) and the bf16 shapes the bf16 matrix-core kernels do not take (widened to fp32
// on the way into LDS, so their probabilities are not rounded either).  Most fp32 up to 128 columns is
// the work of f32x3_step.hip and f32x3_split.hip (f32_route.hip), most short bf16 blocks that of split_mfma.hip.
//
// Measured against kernels with one wavefront per row and serial dot products on the vector ALU: a full
// forward block of 2048 rows, 8 key/value heads for 32, d 128, fp32, 14.6 ms, backward 63, where the split form
// here takes 2.7 backward.
//
// What bounds them: the fp32 matrix cores run at 1/16 of the bf16 rate (64 cycles per
// instruction, 157 TFLOP/s on the chip), so one instruction leaves room for everything that
// feeds it: one LDS read of 4 bytes per lane at most, the softmax in the shadow of the other
// wavefront of the SIMD.  Nothing here is pipelined by hand.
//
// Layouts.  v_mfma_f32_32x32x2_f32, lane = 32 h + n: A element (row n, k = h), B element
// (k = h, column n), C/D register r = (row 8 (r/4) + 4h + r%4, column n).
//  * Products over the head dimension (scores): the order of a contraction is free as long as
//    both operands agree, so columns are taken in groups of 8, half-wave h holding 8g + 4h .. +3
//    of its row: one 16-byte LDS read serves four instructions.
//  * Scores are formed with the OWNED rows as columns (S^T = K Q^T in the query-owning kernels,
//    S = Q K^T in the key-owning one), so register r of a score tile, as it stands, is the B
//    operand (k = h) of the product that contracts over the streamed rows: the A operand is
//    element (row 8 (r/4) + 4h + r%4, column n) of the streamed tile, a conflict-free 4-byte read.
//
// Work split.  A wavefront owns 32 rows.  With enough rows to fill the chip the four wavefronts
// of a workgroup own 128 rows and share every streamed tile (SPLIT = 1); otherwise the workgroup
// owns 32 (64) rows and its wavefronts take the streamed sub-tiles in turn (SPLIT = 4 or 2),
// the partial results meeting in LDS at the end.  Summation orders are fixed: results do not
// depend on timing.
#include "f32_rows.h"
#include "sa_internal.h"

namespace sa {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int WAVES = 4;

// sub-tiles of 32 streamed rows a wavefront takes from one LDS tile
constexpr int subtiles(int SPLIT) { return SPLIT == 1 ? 2 : 1; }
constexpr int tile_rows(int SPLIT) { return 32 * SPLIT * subtiles(SPLIT); }
constexpr int lds_pitch(int DP) { return DP + 4; }          // floats; keeps 16-byte row reads conflict free

__device__ inline f32x16 mfma2(float a, float b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}
__device__ inline f32x16 zero16() {
    f32x16 z;
#pragma unroll
    for (int r = 0; r < 16; ++r) z[r] = 0.f;
    return z;
}

// rows first .. first + ROWS - 1 of a [rows, d] matrix into an LDS tile, zeros beyond row c and
// column d
template <typename T, int DP, int ROWS>
__device__ inline void stage(float* lds, const T* __restrict__ m, int64_t ss, int first, int c, int d) {
    constexpr int CH = DP / 4, N = ROWS * CH / (64 * WAVES);
    float4 x[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int at = (int)threadIdx.x + i * 64 * WAVES, row = at / CH, col = 4 * (at % CH);
        x[i] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (first + row < c && col < d) x[i] = ld4<T>(m + (int64_t)(first + row) * ss + col);
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int at = (int)threadIdx.x + i * 64 * WAVES, row = at / CH, col = 4 * (at % CH);
        *reinterpret_cast<float4*>(lds + row * lds_pitch(DP) + col) = x[i];
    }
}

// an owned row as B operand: group g holds columns 8g + 4h .. + 3
template <typename T, int DP>
__device__ inline void load_row(float4 (&f)[DP / 8], const T* __restrict__ row, int h, int d) {
#pragma unroll
    for (int g = 0; g < DP / 8; ++g) {
        const int col = 8 * g + 4 * h;
        f[g] = col < d ? ld4<T>(row + col) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
}

// 32 x 32 scores: rows = the 32 LDS rows at `rows`, columns = the wavefront's owned rows
template <int DP>
__device__ inline f32x16 scores(const float* rows, const float4 (&f)[DP / 8], int n, int h) {
    f32x16 s = zero16();
    const float* a = rows + n * lds_pitch(DP) + 4 * h;
#pragma unroll
    for (int g = 0; g < DP / 8; ++g) {
        const float4 x = *reinterpret_cast<const float4*>(a + 8 * g);
        s = mfma2(x.x, f[g].x, s);
        s = mfma2(x.y, f[g].y, s);
        s = mfma2(x.z, f[g].z, s);
        s = mfma2(x.w, f[g].w, s);
    }
    return s;
}

// acc[mb] (32 columns of the streamed matrix x owned rows) += streamed^T w
template <int DP, int NB>
__device__ inline void accumulate(f32x16 (&acc)[NB], const float* rows, const f32x16& w, int n, int h) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const float* a = rows + reg_row(r, h) * lds_pitch(DP) + n;
#pragma unroll
        for (int mb = 0; mb < NB; ++mb) acc[mb] = mfma2(a[32 * mb], w[r], acc[mb]);
    }
}

__device__ inline float half_max(float x) { return fmaxf(x, __shfl_xor(x, 32)); }
__device__ inline float half_sum(float x) { return x + __shfl_xor(x, 32); }


// Partial accumulators of the SPLIT wavefronts that own the same rows, summed through LDS
// (wavefront kw keeps column blocks kw, kw + SPLIT, ... of the sum in acc).  buf holds
// SPLIT x 32-row x NB*32-column floats per group of wavefronts.  masks: one word per wavefront of the
// group; returns the rows for which one of them says odd.
template <int SPLIT, int NB>
__device__ inline uint32_t combine(f32x16 (&acc)[NB], float* buf, uint32_t* masks, bool odd, int kw, int lane) {
    const uint32_t own = row_mask(odd);
    if (lane == 0) masks[kw] = own;
    float* mine = buf + kw * NB * 16 * 64;
#pragma unroll
    for (int mb = 0; mb < NB; ++mb)
#pragma unroll
        for (int r = 0; r < 16; ++r) mine[(mb * 16 + r) * 64 + lane] = acc[mb][r];
    __syncthreads();
#pragma unroll
    for (int mb = 0; mb < NB; ++mb) {
        if (mb % SPLIT != kw) continue;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            float x = 0.f;
#pragma unroll
            for (int w = 0; w < SPLIT; ++w) x += buf[((w * NB + mb) * 16 + r) * 64 + lane];
            acc[mb][r] = x;
        }
    }
    uint32_t rows = 0;
#pragma unroll
    for (int w = 0; w < SPLIT; ++w) rows |= masks[w];
    return __builtin_amdgcn_readfirstlane(rows);
}
template <int SPLIT, int DP>
constexpr int tile_floats() { return 2 * tile_rows(SPLIT) * lds_pitch(DP); }

// ------------------------------------------------------------------ forward
template <typename T, int DP, int SPLIT>
__global__ void __launch_bounds__(64 * WAVES, DP > 128 ? 1 : 2)
fwd_f32_kernel(StepArgs p, int n_tiles) {
    constexpr int OWN = WAVES / SPLIT, TK = tile_rows(SPLIT), SUB = subtiles(SPLIT), NB = DP / 32;
    __shared__ __attribute__((aligned(16))) float lds[tile_floats<SPLIT, DP>()];
    __shared__ uint32_t masks[WAVES];
    float* const k_lds = lds;
    float* const v_lds = lds + TK * lds_pitch(DP);

    const int lane = threadIdx.x & 63, n = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int qw = wave / SPLIT, kw = wave % SPLIT;
    int rank, bh, dev_rank;
    decode((int)blockIdx.x, p.B * p.H, rank, bh);
    decode_rank(rank, n_tiles, p.n_q, p.layout, rank, dev_rank);
    const int q0 = (n_tiles - 1 - rank) * 32 * OWN, dev_i = p.n_q - 1 - dev_rank, dev = p.q_dev + dev_i;
    const int b = bh / p.H, hd = bh - b * p.H, d = p.d;
    const int64_t base = b * p.stride_b + hd * p.stride_h + dev_i * p.q_shard;
    const int64_t kv_base = b * p.kv_stride_b + (hd / (p.H / p.H_kv)) * p.kv_stride_h;

    const int a_own = q0 + 32 * qw + n, a = min(a_own, p.c - 1);
    float4 qf[DP / 8];
    load_row<T, DP>(qf, (const T*)p.q + base + (int64_t)a * p.stride_s, h, d);
    f32x16 acc[NB];
#pragma unroll
    for (int mb = 0; mb < NB; ++mb) acc[mb] = zero16();
    float m = -INFINITY, l = 0.f;           // l: this half-wave's share of the row sum

    // the key shards one after the other; contiguous layout: none further on than the queries' own
    const int kv_end = last_shard(p, dev);
    for (int kv = p.kv_dev; kv < kv_end; ++kv) {
        const T* K = (const T*)p.k + kv_base + (kv - p.kv_dev) * p.kv_shard;
        const T* V = (const T*)p.v + kv_base + (kv - p.kv_dev) * p.kv_shard;
        const bool full = block_kind(dev, kv, p.layout) == MASK_FULL;
        const int off = block_off(dev, kv, p.layout);
        const int last_key = full ? p.c - 1 : min(q0 + 32 * OWN, p.c) - 1 - off;          // for the workgroup
        const int wave_last = full ? p.c - 1 : min(q0 + 32 * qw + 31, p.c - 1) - off;     // for the wavefront
        const int lane_last = full ? p.c - 1 : a - off;
        for (int t0 = 0; t0 <= last_key; t0 += TK) {
            __syncthreads();
            stage<T, DP, TK>(k_lds, K, p.kv_stride_s, t0, p.c, d);
            stage<T, DP, TK>(v_lds, V, p.kv_stride_s, t0, p.c, d);
            __syncthreads();
#pragma unroll 1
            for (int s = 0; s < SUB; ++s) {
                const int at = 32 * (SUB * kw + s), key0 = t0 + at;
                if (key0 > wave_last) break;
                f32x16 x = scores<DP>(k_lds + at * lds_pitch(DP), qf, n, h);
                float mx = -INFINITY;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    x[r] = key0 + reg_row(r, h) <= lane_last ? x[r] * p.scale : -INFINITY;
                    mx = fmaxf(mx, x[r]);
                }
                const float m_new = fmaxf(m, half_max(mx));
                const float ref = m_new == -INFINITY ? 0.f : m_new;         // a row without a key so far
                const float alpha = expf(m - ref);
                float sum = 0.f;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    x[r] = expf(x[r] - ref);
                    sum += x[r];
                }
                l = l * alpha + sum;
                if (__builtin_amdgcn_ballot_w64(m_new != m) != 0) {
#pragma unroll
                    for (int mb = 0; mb < NB; ++mb)
#pragma unroll
                        for (int r = 0; r < 16; ++r) acc[mb][r] *= alpha;
                }
                m = m_new;
                accumulate<DP, NB>(acc, v_lds + at * lds_pitch(DP), x, n, h);
            }
        }
    }

    // fold the partial result into the running (O, LSE)
    float l_tot = half_sum(l);
    if (SPLIT > 1) {
        // common reference of the wavefronts that own these rows
        float* const stats = lds;                        // [wave][m | l][32]
        __syncthreads();
        if (h == 0) {
            stats[wave * 64 + n] = m;
            stats[wave * 64 + 32 + n] = l_tot;
        }
        __syncthreads();
        float m_all = -INFINITY;
#pragma unroll
        for (int w = 0; w < SPLIT; ++w) m_all = fmaxf(m_all, stats[(qw * SPLIT + w) * 64 + n]);
        const float ref = m_all == -INFINITY ? 0.f : m_all;
        l_tot = 0.f;
#pragma unroll
        for (int w = 0; w < SPLIT; ++w) {
            const float* sw = stats + (qw * SPLIT + w) * 64;
            l_tot += sw[32 + n] * expf(sw[n] - ref);
        }
        const float f = expf(m - ref);
#pragma unroll
        for (int mb = 0; mb < NB; ++mb)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[mb][r] *= f;
        m = m_all;
        __syncthreads();
    }
    // a row sum that is no positive number although the row sees a key: see f32_rows.h
    const bool odd = a_own < p.c &&
                     (not_finite<NB>(acc) || (!(l_tot > 0.f && l_tot < INFINITY) && sees_a_key(p, dev, a)));
    const uint32_t odd_rows =
        SPLIT > 1 ? combine<SPLIT, NB>(acc, lds + qw * SPLIT * NB * 16 * 64, masks + qw * SPLIT, odd, kw, lane) : row_mask(odd);
    float* L = p.lse + b * p.stat_stride_b + hd * p.stat_stride_h + (int64_t)dev_i * p.c + a;
    const float old = p.fresh ? -INFINITY : *L;
    const float part = l_tot > 0.f ? m + logf(l_tot) : -INFINITY;
    const float top = fmaxf(old, part);
    if (SPLIT > 1) __syncthreads();         // every wavefront has read the old LSE
    // no row here, or no key seen: state unchanged
    if (a_own < p.c && !((odd_rows >> n) & 1) && (part != -INFINITY || p.fresh)) {
        const float ref = top == -INFINITY ? 0.f : top;
        const float w_old = expf(old - ref), w_part = expf(part - ref), w_sum = w_old + w_part;
        const float inv = w_sum > 0.f ? 1.f / w_sum : 0.f;
        const float f_old = w_old * inv, f_part = l_tot > 0.f ? w_part * inv / l_tot : 0.f;
        float* O = p.o + base + (int64_t)a * p.stride_s;
#pragma unroll
        for (int mb = 0; mb < NB; ++mb) {
            if (SPLIT > 1 && mb % SPLIT != kw) continue;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int col = 32 * mb + 8 * g + 4 * h;
                if (col >= d) continue;
                float4* dst = reinterpret_cast<float4*>(O + col);
                float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
                if (f_old != 0.f) {
                    x = *dst;
                    x.x *= f_old; x.y *= f_old; x.z *= f_old; x.w *= f_old;
                }
                x.x = fmaf(acc[mb][4 * g + 0], f_part, x.x); x.y = fmaf(acc[mb][4 * g + 1], f_part, x.y);
                x.z = fmaf(acc[mb][4 * g + 2], f_part, x.z); x.w = fmaf(acc[mb][4 * g + 3], f_part, x.w);
                *dst = x;
            }
        }
        if (kw == 0 && h == 0) *L = top + logf(w_sum);
    }
    each_row<SPLIT>(odd_rows, kw, [&](const StepArgs& again, int i) { fwd_row<T>(again, b, hd, dev_i, q0 + 32 * qw + i, lane); });
}

// scale * acc to 32 owned rows (this lane's row at dst_row), added to what is there unless fresh
template <int SPLIT, int NB>
__device__ inline void add_rows(float* dst_row, const f32x16 (&acc)[NB], float scale, int col0, int d, int kw, int h,
                                bool fresh) {
#pragma unroll
    for (int mb = 0; mb < NB; ++mb) {
        if (SPLIT > 1 && mb % SPLIT != kw) continue;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int col = col0 + 32 * mb + 8 * g + 4 * h;
            if (col >= d) continue;
            float4* dst = reinterpret_cast<float4*>(dst_row + col);
            float4 x = fresh ? make_float4(0.f, 0.f, 0.f, 0.f) : *dst;
            x.x = fmaf(scale, acc[mb][4 * g + 0], x.x); x.y = fmaf(scale, acc[mb][4 * g + 1], x.y);
            x.z = fmaf(scale, acc[mb][4 * g + 2], x.z); x.w = fmaf(scale, acc[mb][4 * g + 3], x.w);
            *dst = x;
        }
    }
}

// ----------------------------------------------------------------------- dQ
template <typename T, int DP, int SPLIT>
__device__ inline void bwd_dq(const StepArgs& p, int n_tiles, int linear, float* lds, uint32_t* masks) {
    constexpr int OWN = WAVES / SPLIT, TK = tile_rows(SPLIT), SUB = subtiles(SPLIT), NB = DP / 32;
    float* const k_lds = lds;
    float* const v_lds = lds + TK * lds_pitch(DP);

    const int lane = threadIdx.x & 63, n = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int qw = wave / SPLIT, kw = wave % SPLIT;
    int rank, bh, dev_rank;
    decode(linear, p.B * p.H, rank, bh);
    decode_rank(rank, n_tiles, p.n_q, p.layout, rank, dev_rank);
    const int q0 = (n_tiles - 1 - rank) * 32 * OWN, dev_i = p.n_q - 1 - dev_rank, dev = p.q_dev + dev_i;
    const int b = bh / p.H, hd = bh - b * p.H, d = p.d;
    const int64_t base = b * p.stride_b + hd * p.stride_h + dev_i * p.q_shard;
    const int64_t kv_base = b * p.kv_stride_b + (hd / (p.H / p.H_kv)) * p.kv_stride_h;
    const int64_t sbase = b * p.stat_stride_b + hd * p.stat_stride_h + (int64_t)dev_i * p.c;

    const int a_own = q0 + 32 * qw + n, a = min(a_own, p.c - 1);
    float4 qf[DP / 8], gf[DP / 8];
    load_row<T, DP>(qf, (const T*)p.q + base + (int64_t)a * p.stride_s, h, d);
    load_row<T, DP>(gf, (const T*)p.dout + base + (int64_t)a * p.stride_s, h, d);
    const float lse = p.lse[sbase + a], delta = p.delta[sbase + a];
    f32x16 acc[NB];
#pragma unroll
    for (int mb = 0; mb < NB; ++mb) acc[mb] = zero16();

    const int kv_end = last_shard(p, dev);
    for (int kv = p.kv_dev; kv < kv_end; ++kv) {
        const T* K = (const T*)p.k + kv_base + (kv - p.kv_dev) * p.kv_shard;
        const T* V = (const T*)p.v + kv_base + (kv - p.kv_dev) * p.kv_shard;
        const bool full = block_kind(dev, kv, p.layout) == MASK_FULL;
        const int off = block_off(dev, kv, p.layout);
        const int last_key = full ? p.c - 1 : min(q0 + 32 * OWN, p.c) - 1 - off;
        const int wave_last = full ? p.c - 1 : min(q0 + 32 * qw + 31, p.c - 1) - off;
        const int lane_last = full ? p.c - 1 : a - off;
        for (int t0 = 0; t0 <= last_key; t0 += TK) {
            __syncthreads();
            stage<T, DP, TK>(k_lds, K, p.kv_stride_s, t0, p.c, d);
            stage<T, DP, TK>(v_lds, V, p.kv_stride_s, t0, p.c, d);
            __syncthreads();
#pragma unroll 1
            for (int s = 0; s < SUB; ++s) {
                const int at = 32 * (SUB * kw + s), key0 = t0 + at;
                if (key0 > wave_last) break;
                f32x16 x = scores<DP>(k_lds + at * lds_pitch(DP), qf, n, h);
                const f32x16 dp = scores<DP>(v_lds + at * lds_pitch(DP), gf, n, h);
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const float pr = key0 + reg_row(r, h) <= lane_last ? expf(x[r] * p.scale - lse) : 0.f;
                    x[r] = pr * (dp[r] - delta);
                }
                accumulate<DP, NB>(acc, k_lds + at * lds_pitch(DP), x, n, h);
            }
        }
    }
    const bool odd = a_own < p.c && not_finite<NB>(acc);
    if (SPLIT > 1) __syncthreads();
    const uint32_t odd_rows =
        SPLIT > 1 ? combine<SPLIT, NB>(acc, lds + qw * SPLIT * NB * 16 * 64, masks + qw * SPLIT, odd, kw, lane) : row_mask(odd);
    if (a_own < p.c && !((odd_rows >> n) & 1))
        add_rows<SPLIT, NB>(p.dq + base + (int64_t)a * p.stride_s, acc, p.scale, 0, d, kw, h, p.fresh);
    each_row<SPLIT>(odd_rows, kw, [&](const StepArgs& again, int i) { dq_row<T>(again, b, hd, dev_i, q0 + 32 * qw + i, lane); });
}

// -------------------------------------------------------------------- dK/dV
// Owned rows are keys, streamed rows queries; the query heads of the group that shares the
// key/value head come one after the other.  DP = 256: a workgroup accumulates one 128-column
// half of dK and dV (both halves beside K and V do not fit the registers) and scores are formed
// once per half.
template <typename T, int DP, int SPLIT>
__device__ inline void bwd_dkdv(const StepArgs& p, int n_tiles, int linear, float* lds, float* stats, uint32_t* masks) {
    constexpr int OWN = WAVES / SPLIT, TK = tile_rows(SPLIT), SUB = subtiles(SPLIT);
    constexpr int HALVES = DP > 128 ? 2 : 1, NB = DP / HALVES / 32;
    float* const q_lds = lds;
    float* const g_lds = lds + TK * lds_pitch(DP);

    const int lane = threadIdx.x & 63, n = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int own = wave / SPLIT, qsub = wave % SPLIT;
    int tile, rest, dev_i;                              // low key tiles see most queries: first
    decode(linear, p.B * p.H_kv * HALVES, tile, rest);
    decode_rank(tile, n_tiles, p.n_kv, p.layout, tile, dev_i);
    const int dev = p.kv_dev + dev_i;
    const int bh = rest / HALVES, col0 = (rest - bh * HALVES) * 128;
    const int k0 = tile * 32 * OWN;
    const int b = bh / p.H_kv, kvh = bh - b * p.H_kv, group = p.H / p.H_kv, d = p.d;
    const int64_t kv_base = b * p.kv_stride_b + kvh * p.kv_stride_h + dev_i * p.kv_shard;

    const int key_own = k0 + 32 * own + n, key = min(key_own, p.c - 1);
    float4 kf[DP / 8], vf[DP / 8];
    load_row<T, DP>(kf, (const T*)p.k + kv_base + (int64_t)key * p.kv_stride_s, h, d);
    load_row<T, DP>(vf, (const T*)p.v + kv_base + (int64_t)key * p.kv_stride_s, h, d);
    f32x16 acck[NB], accv[NB];
#pragma unroll
    for (int mb = 0; mb < NB; ++mb) acck[mb] = accv[mb] = zero16();

    // contiguous layout: earlier devices' queries see nothing of these keys
    const int q_dev0 = p.layout == SA_STRIPED ? p.q_dev : max(p.q_dev, dev);
    for (int member = 0; member < group; ++member) {
        const int hd = kvh * group + member;
        for (int q_dev = q_dev0; q_dev < p.q_dev + p.n_q; ++q_dev) {
            const int64_t base = b * p.stride_b + hd * p.stride_h + (q_dev - p.q_dev) * p.q_shard;
            const int64_t sbase = b * p.stat_stride_b + hd * p.stat_stride_h + (int64_t)(q_dev - p.q_dev) * p.c;
            const T* Q = (const T*)p.q + base;
            const T* G = (const T*)p.dout + base;
            const bool full = block_kind(q_dev, dev, p.layout) == MASK_FULL;
            const int off = block_off(q_dev, dev, p.layout);
            // queries a >= key + off see the key: from this sub-tile on for the workgroup, the wavefront
            const int first_query = full ? 0 : k0 + off;
            const int wave_first = full ? 0 : k0 + 32 * own + off;
            const int lane_first = full ? 0 : key_own + off;
            for (int t0 = first_query / 32 * 32; t0 < p.c; t0 += TK) {
                __syncthreads();
                stage<T, DP, TK>(q_lds, Q, p.stride_s, t0, p.c, d);
                stage<T, DP, TK>(g_lds, G, p.stride_s, t0, p.c, d);
                if (threadIdx.x < 2 * TK) {
                    const int row = min(t0 + (int)threadIdx.x % TK, p.c - 1);
                    stats[threadIdx.x] = threadIdx.x < TK ? p.lse[sbase + row] : p.delta[sbase + row];
                }
                __syncthreads();
#pragma unroll 1
                for (int s = 0; s < SUB; ++s) {
                    const int at = 32 * (SUB * qsub + s), a0 = t0 + at;
                    if (a0 >= p.c) break;
                    if (a0 + 31 < wave_first) continue;
                    const f32x16 x = scores<DP>(q_lds + at * lds_pitch(DP), kf, n, h);
                    f32x16 dp = scores<DP>(g_lds + at * lds_pitch(DP), vf, n, h), pr;
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int row = reg_row(r, h), a = a0 + row;
                        pr[r] = a >= lane_first && a < p.c ? expf(x[r] * p.scale - stats[at + row]) : 0.f;
                        dp[r] = pr[r] * (dp[r] - stats[TK + at + row]);
                    }
                    accumulate<DP, NB>(accv, g_lds + at * lds_pitch(DP) + col0, pr, n, h);
                    accumulate<DP, NB>(acck, q_lds + at * lds_pitch(DP) + col0, dp, n, h);
                }
            }
        }
    }
    const bool odd = key_own < p.c && (not_finite<NB>(accv) || not_finite<NB>(acck));
    uint32_t odd_rows = row_mask(odd);
    if (SPLIT > 1) {
        float* const buf = lds + own * SPLIT * NB * 16 * 64;
        __syncthreads();
        odd_rows = combine<SPLIT, NB>(accv, buf, masks + own * SPLIT, odd, qsub, lane);
        __syncthreads();
        combine<SPLIT, NB>(acck, buf, masks + own * SPLIT, odd, qsub, lane);
    }
    if (key_own < p.c && !((odd_rows >> n) & 1)) {
        const int64_t row = kv_base + (int64_t)key * p.kv_stride_s;
        add_rows<SPLIT, NB>(p.dv + row, accv, 1.f, col0, d, qsub, h, p.fresh);
        add_rows<SPLIT, NB>(p.dk + row, acck, p.scale, col0, d, qsub, h, p.fresh);
    }
    each_row<SPLIT>(odd_rows, qsub, [&](const StepArgs& again, int i) {
        dkdv_row<T>(again, b, kvh, dev_i, k0 + 32 * own + i, col0, HALVES > 1 ? min(d, col0 + 128) : d, lane);
    });
}

// Both in one launch (KEYS and QUERIES): workgroups 0 .. n_dkdv - 1 own keys, the others queries.
// They share nothing but the inputs; where neither fills the chip they run beside each other, and
// a step is one launch less.  At 256 columns each by itself: together they spill registers.
template <typename T, int DP, int SPLIT, bool KEYS, bool QUERIES>
__global__ void __launch_bounds__(64 * WAVES, DP > 64 ? 1 : 2)
bwd_f32_kernel(StepArgs p, int n_tiles, int n_dkdv) {
    __shared__ __attribute__((aligned(16))) float lds[tile_floats<SPLIT, DP>()];
    __shared__ float stats[KEYS ? 2 * tile_rows(SPLIT) : 1];        // LSE | delta of a tile's queries
    __shared__ uint32_t masks[WAVES];
    if (KEYS && (!QUERIES || (int)blockIdx.x < n_dkdv))
        bwd_dkdv<T, DP, SPLIT>(p, n_tiles, (int)blockIdx.x, lds, stats, masks);
    else if (QUERIES) bwd_dq<T, DP, SPLIT>(p, n_tiles, (int)blockIdx.x - (KEYS ? n_dkdv : 0), lds, masks);
}

// ----------------------------------------------------------------- dispatch
template <typename T, int DP, int SPLIT>
hipError_t run_fwd(const StepArgs& a, hipStream_t st) {
    const int rows = 32 * (WAVES / SPLIT), n_tiles = (a.c + rows - 1) / rows;
    hipLaunchKernelGGL((fwd_f32_kernel<T, DP, SPLIT>), dim3((unsigned)n_tiles * a.n_q * a.B * a.H), dim3(64 * WAVES),
                       0, st, a, n_tiles);
    return hipGetLastError();
}
template <typename T, int DP, int SPLIT>
hipError_t run_bwd(const StepArgs& a, hipStream_t st) {
    const int rows = 32 * (WAVES / SPLIT), n_tiles = (a.c + rows - 1) / rows;
    const int n_dkdv = n_tiles * a.n_kv * a.B * a.H_kv * (DP > 128 ? 2 : 1), n_dq = n_tiles * a.n_q * a.B * a.H;
    const dim3 block(64 * WAVES);
    if constexpr (DP <= 128) {
        hipLaunchKernelGGL((bwd_f32_kernel<T, DP, SPLIT, true, true>), dim3((unsigned)(n_dkdv + n_dq)), block, 0, st, a,
                           n_tiles, n_dkdv);
    } else {
        hipLaunchKernelGGL((bwd_f32_kernel<T, DP, SPLIT, false, true>), dim3((unsigned)n_dq), block, 0, st, a, n_tiles,
                           0);
        if (hipError_t e = hipGetLastError()) return e;
        hipLaunchKernelGGL((bwd_f32_kernel<T, DP, SPLIT, true, false>), dim3((unsigned)n_dkdv), block, 0, st, a,
                           n_tiles, n_dkdv);
    }
    return hipGetLastError();
}

template <typename T, int DP>
hipError_t run(const StepArgs& a, bool backward, hipStream_t st) {
    constexpr int MOST = DP > 128 ? 2 : 4;          // what 160 KiB of LDS hold
    const bool split = few_row_tiles(a, backward);
    if (backward) return split ? run_bwd<T, DP, MOST>(a, st) : run_bwd<T, DP, 1>(a, st);
    return split ? run_fwd<T, DP, MOST>(a, st) : run_fwd<T, DP, 1>(a, st);
}
hipError_t run(const StepArgs& a, int dtype, bool backward, hipStream_t st) {
    if (dtype == SA_F32) return run<float, 256>(a, backward, st);
    if (a.d <= 32) return run<__hip_bfloat16, 32>(a, backward, st);
    if (a.d <= 64) return run<__hip_bfloat16, 64>(a, backward, st);
    if (a.d <= 128) return run<__hip_bfloat16, 128>(a, backward, st);
    return run<__hip_bfloat16, 256>(a, backward, st);
}
// fp32 launches of few row tiles
template <int DP>
hipError_t run_few(const StepArgs& a, bool backward, hipStream_t st) {
    return backward ? run_bwd<float, DP, 4>(a, st) : run_fwd<float, DP, 4>(a, st);
}
hipError_t launch_f32_storage(const StepArgs& a, bool backward, hipStream_t st) {
    const F32Route route = f32_route(a, backward);
    if (route == F32_SPLIT) return launch_f32x3_split(a, backward, st);
    if (route != F32_INSTRUCTION) return launch_f32x3(a, backward, route == F32_TERMS_ALONE, st);
    return a.d <= 32 ? run_few<32>(a, backward, st) : a.d <= 64 ? run_few<64>(a, backward, st) : run_few<128>(a, backward, st);
}

}  // namespace

hipError_t launch_fwd_f32(const StepArgs& a, int dtype, hipStream_t st) {
    if (few_rows_wanted(a, dtype, false)) return launch_few_rows(a, dtype, false, st);
    if (dtype == SA_F32 && a.d <= 128) return launch_f32_storage(a, false, st);
    if (short_exact_wanted(a, dtype, false)) return launch_short_exact(a, false, st);
    return run(a, dtype, false, st);
}
hipError_t launch_bwd_f32(const StepArgs& a, int dtype, hipStream_t st) {
    if (few_rows_wanted(a, dtype, true)) return launch_few_rows(a, dtype, true, st);
    if (dtype == SA_F32 && a.d <= 128) return launch_f32_storage(a, true, st);
    if (short_exact_wanted(a, dtype, true)) return launch_short_exact(a, true, st);
    return run(a, dtype, true, st);
}

}  // namespace sa
