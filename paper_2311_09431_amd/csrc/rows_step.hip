// Ring steps on blocks of a few rows, in plain fp32 arithmetic: a group of 16, 32 or 64 lanes owns a row
// (up to 64, 128, 256 columns, four a lane), looks at the allowed pairs only and sums products over
// its lanes.
//
// What bounds such a step is one launch and a few dependent memory round trips.  The matrix-core kernels
// give every (batch, head) a workgroup of 32 or 128 rows with tile buffers for one or two workgroups per
// compute unit, so a block of one row and 512 heads took 17 us forward and 31 us backward (bf16, d 100),
// where this takes 8 and 8.6 us.  Figures at few_rows_wanted.
#include "f32_rows.h"
#include "sa_internal.h"

namespace sa {

namespace {

template <int LANES>
__device__ inline float group_sum(float x) {
#pragma unroll
    for (int o = LANES / 2; o > 0; o >>= 1) x += __shfl_xor(x, o);
    return x;
}
__device__ inline float dot4(float4 a, float4 b) { return fmaf(a.w, b.w, fmaf(a.z, b.z, fmaf(a.y, b.y, a.x * b.x))); }
__device__ inline void add4(float4& acc, float w, float4 x) {
    acc.x = fmaf(w, x.x, acc.x); acc.y = fmaf(w, x.y, acc.y);
    acc.z = fmaf(w, x.z, acc.z); acc.w = fmaf(w, x.w, acc.w);
}
template <typename T>
__device__ inline float4 cols(const T* row, int col, int d) {
    return col < d ? ld4<T>(row + col) : make_float4(0.f, 0.f, 0.f, 0.f);
}

// row a of (batch, head) bh, from the number of a lane group; false: none
__device__ inline bool own_row(int group, int c, int n_bh, int& a, int& bh) {
    bh = group / c;
    a = group - bh * c;
    return bh < n_bh;
}
template <int LANES>
__device__ inline int group_number(int block) { return block * (256 / LANES) + (int)threadIdx.x / LANES; }

template <typename T, int LANES>
__global__ void __launch_bounds__(256)
fwd_rows_kernel(StepArgs p) {
    int a, bh;
    if (!own_row(group_number<LANES>((int)blockIdx.x), p.c, p.B * p.H, a, bh)) return;
    const int keys = block_kind(p.q_dev, p.kv_dev, p.layout) == MASK_FULL ? p.c
                                                                          : a - block_off(p.q_dev, p.kv_dev, p.layout) + 1;
    if (keys <= 0) return;                                  // state unchanged
    const int b = bh / p.H, hd = bh - b * p.H, d = p.d, col = 4 * ((int)threadIdx.x % LANES);
    const int64_t row = b * p.stride_b + hd * p.stride_h + (int64_t)a * p.stride_s;
    const int64_t kv = b * p.kv_stride_b + (hd / (p.H / p.H_kv)) * p.kv_stride_h;
    const float4 q = cols<T>((const T*)p.q + row, col, d);
    float* const O = p.o + row + col;
    float* const L = p.lse + b * p.stat_stride_b + hd * p.stat_stride_h + a;
    // running state: weight exp(lse) with l = 1 (or nothing yet)
    float m = *L, l = m == -INFINITY ? 0.f : 1.f;
    const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
    const float4 old = col < d ? *reinterpret_cast<const float4*>(O) : zero;
    float4 acc = l != 0.f ? old : zero;
    for (int k = 0; k < keys; ++k) {
        const int64_t at = kv + (int64_t)k * p.kv_stride_s;
        const float4 kr = cols<T>((const T*)p.k + at, col, d), vr = cols<T>((const T*)p.v + at, col, d);
        const float s = p.scale * group_sum<LANES>(dot4(q, kr));
        const float m_new = fmaxf(m, s), ref = m_new == -INFINITY ? 0.f : m_new;
        const float alpha = m == -INFINITY ? 0.f : expf(m - m_new), pr = expf(s - ref);
        l = l * alpha + pr;
        acc.x *= alpha; acc.y *= alpha; acc.z *= alpha; acc.w *= alpha;
        add4(acc, pr, vr);
        m = m_new;
    }
    // every key it sees at -inf, and no state: no number, as in f32_rows.h
    const float inv = 1.f / l;
    if (col < d) *reinterpret_cast<float4*>(O) = make_float4(acc.x * inv, acc.y * inv, acc.z * inv, acc.w * inv);
    if (col == 0) *L = l == 0.f ? NAN : m + logf(l);
}

// groups 0 .. n_keys - 1 own key rows, the others query rows
template <typename T, int LANES>
__global__ void __launch_bounds__(256)
bwd_rows_kernel(StepArgs p, int key_blocks) {
    const int d = p.d, col = 4 * ((int)threadIdx.x % LANES), share = p.H / p.H_kv;
    const bool full = block_kind(p.q_dev, p.kv_dev, p.layout) == MASK_FULL;
    const int off = block_off(p.q_dev, p.kv_dev, p.layout);
    int a, bh;
    if ((int)blockIdx.x < key_blocks) {
        if (!own_row(group_number<LANES>((int)blockIdx.x), p.c, p.B * p.H_kv, a, bh)) return;
        const int b = bh / p.H_kv, kvh = bh - b * p.H_kv;
        const int64_t row = b * p.kv_stride_b + kvh * p.kv_stride_h + (int64_t)a * p.kv_stride_s;
        const float4 kr = cols<T>((const T*)p.k + row, col, d), vr = cols<T>((const T*)p.v + row, col, d);
        float4 dk = make_float4(0.f, 0.f, 0.f, 0.f), dv = dk;
        for (int member = 0; member < share; ++member) {
            const int hd = kvh * share + member;
            const int64_t base = b * p.stride_b + hd * p.stride_h, stat = b * p.stat_stride_b + hd * p.stat_stride_h;
            for (int i = full ? 0 : a + off; i < p.c; ++i) {
                const int64_t at = base + (int64_t)i * p.stride_s;
                const float4 q = cols<T>((const T*)p.q + at, col, d), g = cols<T>((const T*)p.dout + at, col, d);
                const float pr = expf(p.scale * group_sum<LANES>(dot4(q, kr)) - p.lse[stat + i]);
                const float ds = pr * (group_sum<LANES>(dot4(g, vr)) - p.delta[stat + i]);
                add4(dv, pr, g);
                add4(dk, ds, q);
            }
        }
        if (col >= d) return;
        float4* const DV = reinterpret_cast<float4*>(p.dv + row + col);
        float4* const DK = reinterpret_cast<float4*>(p.dk + row + col);
        float4 x = *DV, y = *DK;
        x.x += dv.x; x.y += dv.y; x.z += dv.z; x.w += dv.w;
        add4(y, p.scale, dk);
        *DV = x;
        *DK = y;
        return;
    }
    if (!own_row(group_number<LANES>((int)blockIdx.x - key_blocks), p.c, p.B * p.H, a, bh)) return;
    const int b = bh / p.H, hd = bh - b * p.H, keys = full ? p.c : a - off + 1;
    const int64_t row = b * p.stride_b + hd * p.stride_h + (int64_t)a * p.stride_s;
    const int64_t kv = b * p.kv_stride_b + (hd / share) * p.kv_stride_h;
    const float4 q = cols<T>((const T*)p.q + row, col, d), g = cols<T>((const T*)p.dout + row, col, d);
    const int64_t stat = b * p.stat_stride_b + hd * p.stat_stride_h + a;
    const float lse = p.lse[stat], delta = p.delta[stat];
    float4 dq = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int k = 0; k < keys; ++k) {
        const int64_t at = kv + (int64_t)k * p.kv_stride_s;
        const float4 kr = cols<T>((const T*)p.k + at, col, d), vr = cols<T>((const T*)p.v + at, col, d);
        const float pr = expf(p.scale * group_sum<LANES>(dot4(q, kr)) - lse);
        add4(dq, pr * (group_sum<LANES>(dot4(g, vr)) - delta), kr);
    }
    if (col >= d) return;
    float4* const DQ = reinterpret_cast<float4*>(p.dq + row + col);
    float4 x = *DQ;
    add4(x, p.scale, dq);
    *DQ = x;
}

template <typename T, int LANES>
hipError_t run(const StepArgs& a, bool backward, hipStream_t st) {
    const auto blocks = [&](int heads) { return (int)(((int64_t)a.c * a.B * heads * LANES + 255) / 256); };
    if (backward)
        hipLaunchKernelGGL((bwd_rows_kernel<T, LANES>), dim3(blocks(a.H_kv) + blocks(a.H)), dim3(256), 0, st, a,
                           blocks(a.H_kv));
    else hipLaunchKernelGGL((fwd_rows_kernel<T, LANES>), dim3(blocks(a.H)), dim3(256), 0, st, a);
    return hipGetLastError();
}
template <typename T>
hipError_t run(const StepArgs& a, bool backward, hipStream_t st) {
    if (a.d <= 64) return run<T, 16>(a, backward, st);
    return a.d <= 128 ? run<T, 32>(a, backward, st) : run<T, 64>(a, backward, st);
}

}  // namespace

// Up to 8 rows, or 16 where the other kernels are the fp32 ones (fp32 storage, more than 128 columns); in
// the backward a key row meets the queries of its whole group one after the other, at most 16 then.
// Single steps, us, here / those kernels: bf16, d 64, 8 rows, 32 heads forward 8.1 / 9.0, backward 8.8 /
// 8.6, 512 heads 8.0 / 11.7 and 8.7 / 17.9; d 100 8.1 / 10.7, 8.6 / 10.4, 9.2 / 17.8, 8.8 / 34.1; 16 rows, d 64,
// 32 heads 11.5 / 9.1; 32 query heads on 8, 8 rows, d 64, backward (32 queries a key) 16.4 / 11.2.  fp32,
// 16 rows: d 64 9.1 / 9.1, 9.3 / 11.4, 9.9 / 14.4, 10.4 / 32.9, 24 rows 11.9 / 9.1 forward; d 128 9.9 / 12.6,
// 9.4 / 18.9, 11.4 / 25.2, 17 / 56.  bf16, d 256, 16 rows 12.3 / 25.3, 11.7 / 77, 22 / 51, 31 / 259.  (8 us is what
// a launch costs in this series of launches.)
bool few_rows_wanted(const StepArgs& a, int dtype, bool backward) {
    const int most = dtype == SA_F32 || a.d > 128 ? 16 : 8;
    return a.c <= most && a.n_q == 1 && a.n_kv == 1 && !a.fresh && (!backward || a.c * (a.H / a.H_kv) <= 16);
}
hipError_t launch_few_rows(const StepArgs& a, int dtype, bool backward, hipStream_t st) {
    return dtype == SA_F32 ? run<float>(a, backward, st) : run<__hip_bfloat16>(a, backward, st);
}

}  // namespace sa
