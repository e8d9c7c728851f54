// Single rows of a ring step in plain fp32 arithmetic, one wavefront a row, looking at nothing but
// the pairs that the mask allows.
//
// A row whose sum of weights in the fp32-precision matrix-core kernels (f32_step.hip, f32x3_step.hip,
// the exact ones of split_mfma.hip) is no positive number although it sees a key, has a NaN or +inf
// score, nothing but scores of -inf, or scores that overflow a reference: a kernel looks there once,
// at its end, and does such a row over here.  One wavefront and serial dot products: about the speed
// of a vector kernel, and only for such rows.
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

// one past the last key shard that device dev's queries see
__device__ inline int last_shard(const StepArgs& p, int dev) {
    return p.layout == SA_STRIPED ? p.kv_dev + p.n_kv : min(p.kv_dev + p.n_kv, dev + 1);
}
// whether row a of device dev sees a key in this launch's blocks
__device__ inline bool sees_a_key(const StepArgs& p, int dev, int a) {
    return p.layout != SA_STRIPED || a > 0 || p.kv_dev <= dev;
}

// rows (bit n: lanes n and n + 32) for which a lane says so
__device__ inline uint32_t row_mask(bool lane_says) {
    const uint64_t m = __builtin_amdgcn_ballot_w64(lane_says);
    return (uint32_t)m | (uint32_t)(m >> 32);
}

// the rows set in a mask, taken in turn by the SPLIT wavefronts that own them
template <int SPLIT, typename Row>
__device__ inline void each_row(uint32_t rows, int wave, Row row) {
#pragma unroll 1
    for (; rows != 0; rows &= rows - 1) {
        const int n = __builtin_ctz(rows);
        if (n % SPLIT == wave) row(n);
    }
}

// columns lane, lane + 64, ... of a row
constexpr int ROW_COLS = 256 / 64;

template <typename T>
__device__ inline float dot_rows(const T* x, const T* y, int d) {
    float s = 0.f;
#pragma unroll 1
    for (int t = 0; t < d; t += 4) {
        const float4 a = ld4<T>(x + t), b = ld4<T>(y + t);
        s = fmaf(a.x, b.x, s);
        s = fmaf(a.y, b.y, s);
        s = fmaf(a.z, b.z, s);
        s = fmaf(a.w, b.w, s);
    }
    return s;
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
#pragma unroll 1
    for (int i = 0; i < n; ++i) {
        const float w = __shfl(weight, i);
#pragma unroll
        for (int k = 0; k < ROW_COLS; ++k) {
            const int col = col0 + lane + 64 * k;
            if (col < d) acc[k] = fmaf(w, ld1(rows + i * ss + col), acc[k]);
        }
    }
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

}  // namespace sa
