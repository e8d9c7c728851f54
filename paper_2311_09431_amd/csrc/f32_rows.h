// Single rows of a ring step in plain fp32 arithmetic, one wavefront a row, looking at nothing but
// the pairs that the mask allows.
//
// The fp32-precision matrix-core kernels (f32_step.hip, f32x3_step.hip, the exact ones of
// split_mfma.hip) multiply whole 32 x 32 sub-tiles, masked pairs with a weight of zero, and two of
// them an operand as three terms.  For finite numbers that is the same sum; an infinite or NaN element
// makes 0 * inf, inf - inf, or a sum of row weights that is no number.  All of these leave something
// that is not finite in the row's accumulators or row sum, so a kernel looks there once, at its end,
// and a row where it finds it is done over here: NaN and infinities then reach the rows that see them
// and no others.  Rows too small for three terms go the same way (FAINT).  One wavefront and serial dot products: about the
// speed of a vector kernel, and only for such rows.  The looks cost 16 fmas and 16 maxima per 32 x 32 accumulator and
// workgroup.
#pragma once
#include <hip/hip_bf16.h>

#include "sa_internal.h"

namespace sa {

template <typename T>
__device__ inline float4 ld4(const T* p);
template <>
__device__ inline float4 ld4<float>(const float* p) { return *reinterpret_cast<const float4*>(p); }
template <>
__device__ inline float4 ld4<__hip_bfloat16>(const __hip_bfloat16* p) {
    const uint2 raw = *reinterpret_cast<const uint2*>(p);
    return make_float4(__uint_as_float(raw.x << 16), __uint_as_float(raw.x & 0xffff0000u),
                       __uint_as_float(raw.y << 16), __uint_as_float(raw.y & 0xffff0000u));
}
__device__ inline float ld1(const float* p) { return *p; }
__device__ inline float ld1(const __hip_bfloat16* p) {
    return __uint_as_float((uint32_t)(*reinterpret_cast<const uint16_t*>(p)) << 16);
}

// What f32_step.hip, f32x3_step.hip and split_mfma.hip share beside that.

// streamed row (within a 32-row sub-tile) of register r of a 32 x 32 score tile, h = lane / 32
__device__ inline int reg_row(int r, int h) { return 8 * (r / 4) + 4 * h + r % 4; }
// Workgroup -> (tile rank, head): ranks heaviest first over all heads.
__device__ inline void decode(int linear, int n_heads, int& rank, int& head) {
    rank = linear / n_heads;
    head = linear - rank * n_heads;
}
// one past the last key shard that device dev's queries see
__device__ inline int last_shard(const StepArgs& p, int dev) {
    return p.layout == SA_STRIPED ? p.kv_dev + p.n_kv : min(p.kv_dev + p.n_kv, dev + 1);
}
// whether row a of device dev sees a key in this launch's blocks
__device__ inline bool sees_a_key(const StepArgs& p, int dev, int a) {
    return p.layout != SA_STRIPED || a > 0 || p.kv_dev <= dev;
}

// some register of the first NB accumulators is infinite or NaN
template <int NB, typename Acc>
__device__ inline bool not_finite(const Acc& acc) {
    float z[4] = {0.f, 0.f, 0.f, 0.f};          // four chains: one would wait for itself
#pragma unroll
    for (int mb = 0; mb < NB; ++mb)
#pragma unroll
        for (int r = 0; r < 16; ++r) z[r % 4] = fmaf(acc[mb][r], 0.f, z[r % 4]);
    return (z[0] + z[1]) + (z[2] + z[3]) != 0.f;
}
// The largest magnitude in the first NB accumulators (NaN passed over).  Three bf16 terms cover a number down to 2^-109;
// below, the last one is subnormal and up to 2^-134 is lost of it.  So where operands are such terms and the results of all 32
// rows of a tile are below FAINT, those that are not all zero are done over here too; from FAINT on what is lost is below
// fp32's own rounding, 2^-24 of the tile's largest row, for weights and elements whose squares sum to less than 2^10 over
// the row.  (Faint rows beside a louder one are what peaked scores leave: keys whose every probability is that small, and
// no operand.  Done over, each by itself, they cost 8 heads of 2048 rows, d 64, scores of standard deviation 300, 1.64 ms
// backward instead of 0.12, of 50 0.49.)  dO, V, K or Q scaled by 2^-100 to 2^-120, heads of 257 to 512 rows, the worst
// output's error against 64 bits: terms alone 4.6e-4, the fp32 instruction 5.0e-7, done over 3.2e-7.  (Where every product has a factor below 2^-134, the result is
// zero: it is below fp32's normal numbers but for factors beyond 2^8.)
constexpr float FAINT = 0x1p-105f;
template <int NB, typename Acc>
__device__ inline float loudest(const Acc& acc) {
    float z[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int mb = 0; mb < NB; ++mb)
#pragma unroll
        for (int r = 0; r < 16; ++r) z[r % 4] = fmaxf(z[r % 4], fabsf(acc[mb][r]));
    return fmaxf(fmaxf(z[0], z[1]), fmaxf(z[2], z[3]));
}
// rows (bit n: lanes n and n + 32) for which a lane says so
__device__ inline uint32_t row_mask(bool lane_says) {
    const uint64_t m = __builtin_amdgcn_ballot_w64(lane_says);
    return (uint32_t)m | (uint32_t)(m >> 32);
}
// the rows in the shard that are not all zero, if all are faint
__device__ inline uint32_t faint_rows(float top, bool in_shard) {
    return row_mask(top >= FAINT) ? 0 : row_mask(in_shard && top > 0.f);
}

// The rows set in a mask, taken in turn by the SPLIT wavefronts that own them: row(arguments, n).  The
// launch's arguments (a kernel's first parameter) are read anew for it, so that none of them has to
// be kept until here by the kernel's ordinary course (scalar registers spilled in its loops
// otherwise: a backward step of 32 query heads on 8, 6 rows, d 100, 18.6 against 15.6 us).
__device__ inline const StepArgs& launch_args() {
    typedef const StepArgs __attribute__((address_space(4))) Arguments;
    Arguments* at = (Arguments*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(at));
    return *(const StepArgs*)at;
}
template <int SPLIT, typename Row>
__device__ inline void each_row(uint32_t rows, int wave, Row row) {
    if (rows == 0) return;
    const StepArgs& p = launch_args();
#pragma unroll 1
    for (; rows != 0; rows &= rows - 1) {
        const int n = __builtin_ctz(rows);
        if (n % SPLIT == wave) row(p, n);
    }
}

// columns lane, lane + 64, ... of a row
constexpr int ROW_COLS = 256 / 64;

template <typename T>
__device__ inline float dot_rows(const T* x, const T* y, int d) {
    double s = 0.;          // (sums in fp64: a row done over is no further off than the kernels' own)
#pragma unroll 1
    for (int t = 0; t < d; t += 4) {
        const float4 a = ld4<T>(x + t), b = ld4<T>(y + t);
        s = fma((double)a.x, (double)b.x, s);
        s = fma((double)a.y, (double)b.y, s);
        s = fma((double)a.z, (double)b.z, s);
        s = fma((double)a.w, (double)b.w, s);
    }
    return (float)s;
}
__device__ inline float wave_max(float x) {
#pragma unroll 1
    for (int o = 32; o > 0; o >>= 1) x = fmaxf(x, __shfl_xor(x, o));
    return x;
}
__device__ inline float wave_sum(float x) {
#pragma unroll 1
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
    return x;
}
// acc += sum over n rows of rows' weights (lane i holds row i's)
template <typename T>
__device__ inline void add_weighted(float (&acc)[ROW_COLS], float weight, const T* rows, int64_t ss, int n, int col0,
                                    int d, int lane) {
    double part[ROW_COLS] = {};
#pragma unroll 1
    for (int i = 0; i < n; ++i) {
        const float w = __shfl(weight, i);
#pragma unroll
        for (int k = 0; k < ROW_COLS; ++k) {
            const int col = col0 + lane + 64 * k;
            if (col < d) part[k] = fma((double)w, (double)ld1(rows + i * ss + col), part[k]);
        }
    }
#pragma unroll
    for (int k = 0; k < ROW_COLS; ++k) acc[k] += (float)part[k];
}

// forward, query row a of the launch's device dev_i: its shards folded into (O, LSE)
template <typename T>
__device__ inline void fwd_row(const StepArgs& p, int b, int hd, int dev_i, int a, int lane) {
    const int dev = p.q_dev + dev_i;
    const int64_t row = b * p.stride_b + hd * p.stride_h + dev_i * p.q_shard + (int64_t)a * p.stride_s;
    const int64_t kv_base = b * p.kv_stride_b + (hd / (p.H / p.H_kv)) * p.kv_stride_h;
    const T* q = (const T*)p.q + row;
    float* O = p.o + row;
    float* L = p.lse + b * p.stat_stride_b + hd * p.stat_stride_h + (int64_t)dev_i * p.c + a;
    const bool sees = sees_a_key(p, dev, a);
    if (!sees && !p.fresh) return;                          // state unchanged
    // running state: weight exp(lse) with l = 1 (or nothing yet)
    float m = p.fresh ? -INFINITY : *L, l = m == -INFINITY ? 0.f : 1.f, acc[ROW_COLS];
#pragma unroll
    for (int k = 0; k < ROW_COLS; ++k) acc[k] = l != 0.f && lane + 64 * k < p.d ? O[lane + 64 * k] : 0.f;
    const int kv_end = last_shard(p, dev);
#pragma unroll 1
    for (int kv = p.kv_dev; kv < kv_end; ++kv) {
        const T* K = (const T*)p.k + kv_base + (kv - p.kv_dev) * p.kv_shard;
        const T* V = (const T*)p.v + kv_base + (kv - p.kv_dev) * p.kv_shard;
        const int keys = block_kind(dev, kv, p.layout) == MASK_FULL ? p.c : a - block_off(dev, kv, p.layout) + 1;
#pragma unroll 1
        for (int k0 = 0; k0 < keys; k0 += 64) {
            const bool valid = k0 + lane < keys;
            const float s = valid ? p.scale * dot_rows<T>(q, K + (int64_t)(k0 + lane) * p.kv_stride_s, p.d) : -INFINITY;
            const float m_new = fmaxf(m, wave_max(s)), ref = m_new == -INFINITY ? 0.f : m_new;
            const float alpha = m == -INFINITY ? 0.f : expf(m - m_new);
            const float pr = valid ? expf(s - ref) : 0.f;
            l = l * alpha + wave_sum(pr);
#pragma unroll
            for (int k = 0; k < ROW_COLS; ++k) acc[k] *= alpha;
            add_weighted<T>(acc, pr, V + (int64_t)k0 * p.kv_stride_s, p.kv_stride_s, min(64, keys - k0), 0, p.d, lane);
            m = m_new;
        }
    }
    // every key it sees at -inf, and no state: the softmax of nothing but zeros is no number
    const float inv = sees ? 1.f / l : 0.f;
#pragma unroll
    for (int k = 0; k < ROW_COLS; ++k)
        if (lane + 64 * k < p.d) O[lane + 64 * k] = acc[k] * inv;
    if (lane == 0) *L = !sees ? -INFINITY : l == 0.f ? NAN : m + logf(l);
}

// backward, query row a of the launch's device dev_i: adds to (fresh: stores) its dQ
template <typename T>
__device__ inline void dq_row(const StepArgs& p, int b, int hd, int dev_i, int a, int lane) {
    const int dev = p.q_dev + dev_i;
    const int64_t row = b * p.stride_b + hd * p.stride_h + dev_i * p.q_shard + (int64_t)a * p.stride_s;
    const int64_t kv_base = b * p.kv_stride_b + (hd / (p.H / p.H_kv)) * p.kv_stride_h;
    const int64_t stat = b * p.stat_stride_b + hd * p.stat_stride_h + (int64_t)dev_i * p.c + a;
    const T* q = (const T*)p.q + row;
    const T* g = (const T*)p.dout + row;
    const float lse = p.lse[stat], delta = p.delta[stat];
    float acc[ROW_COLS] = {};
    const int kv_end = last_shard(p, dev);
#pragma unroll 1
    for (int kv = p.kv_dev; kv < kv_end; ++kv) {
        const T* K = (const T*)p.k + kv_base + (kv - p.kv_dev) * p.kv_shard;
        const T* V = (const T*)p.v + kv_base + (kv - p.kv_dev) * p.kv_shard;
        const int keys = block_kind(dev, kv, p.layout) == MASK_FULL ? p.c : a - block_off(dev, kv, p.layout) + 1;
#pragma unroll 1
        for (int k0 = 0; k0 < keys; k0 += 64) {
            float ds = 0.f;
            if (k0 + lane < keys) {
                const int64_t at = (int64_t)(k0 + lane) * p.kv_stride_s;
                const float pr = expf(p.scale * dot_rows<T>(q, K + at, p.d) - lse);
                ds = pr * (dot_rows<T>(g, V + at, p.d) - delta);
            }
            add_weighted<T>(acc, ds, K + (int64_t)k0 * p.kv_stride_s, p.kv_stride_s, min(64, keys - k0), 0, p.d, lane);
        }
    }
    float* DQ = p.dq + row;
#pragma unroll
    for (int k = 0; k < ROW_COLS; ++k)
        if (lane + 64 * k < p.d) DQ[lane + 64 * k] = (p.fresh ? 0.f : DQ[lane + 64 * k]) + p.scale * acc[k];
}

// backward, key row `key` of the launch's device dev_i: adds to (fresh: stores) columns col0 .. end - 1 of
// its dK and dV
template <typename T>
__device__ inline void dkdv_row(const StepArgs& p, int b, int kvh, int dev_i, int key, int col0, int end, int lane) {
    const int dev = p.kv_dev + dev_i, group = p.H / p.H_kv;
    const int64_t row = b * p.kv_stride_b + kvh * p.kv_stride_h + dev_i * p.kv_shard + (int64_t)key * p.kv_stride_s;
    const T* kr = (const T*)p.k + row;
    const T* vr = (const T*)p.v + row;
    float acck[ROW_COLS] = {}, accv[ROW_COLS] = {};
    const int q_dev0 = p.layout == SA_STRIPED ? p.q_dev : max(p.q_dev, dev);
#pragma unroll 1
    for (int member = 0; member < group; ++member) {
        const int hd = kvh * group + member;
#pragma unroll 1
        for (int q_dev = q_dev0; q_dev < p.q_dev + p.n_q; ++q_dev) {
            const int64_t base = b * p.stride_b + hd * p.stride_h + (q_dev - p.q_dev) * p.q_shard;
            const int64_t sbase = b * p.stat_stride_b + hd * p.stat_stride_h + (int64_t)(q_dev - p.q_dev) * p.c;
            const T* Q = (const T*)p.q + base;
            const T* G = (const T*)p.dout + base;
            const int first = block_kind(q_dev, dev, p.layout) == MASK_FULL ? 0 : key + block_off(q_dev, dev, p.layout);
#pragma unroll 1
            for (int a0 = first; a0 < p.c; a0 += 64) {
                float pr = 0.f, ds = 0.f;
                if (a0 + lane < p.c) {
                    const int64_t at = (int64_t)(a0 + lane) * p.stride_s;
                    pr = expf(p.scale * dot_rows<T>(kr, Q + at, p.d) - p.lse[sbase + a0 + lane]);
                    ds = pr * (dot_rows<T>(vr, G + at, p.d) - p.delta[sbase + a0 + lane]);
                }
                const int rows = min(64, p.c - a0);
                add_weighted<T>(accv, pr, G + (int64_t)a0 * p.stride_s, p.stride_s, rows, col0, end, lane);
                add_weighted<T>(acck, ds, Q + (int64_t)a0 * p.stride_s, p.stride_s, rows, col0, end, lane);
            }
        }
    }
#pragma unroll
    for (int k = 0; k < ROW_COLS; ++k) {
        const int col = col0 + lane + 64 * k;
        if (col >= end) continue;
        p.dv[row + col] = (p.fresh ? 0.f : p.dv[row + col]) + accv[k];
        p.dk[row + col] = (p.fresh ? 0.f : p.dk[row + col]) + p.scale * acck[k];
    }
}

}  // namespace sa
