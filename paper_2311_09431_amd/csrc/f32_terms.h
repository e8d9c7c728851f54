// fp32 numbers on the bf16 matrix cores: three bf16 terms, and exponentials whose argument is formed
// with fp32's own rounding.
#pragma once
#include "mfma_tiles.h"

namespace sa {

// x = hi + mid + lo (+ less than 2^-26 x; below 2^-109 in magnitude lo is a subnormal number, and x has
// fewer than 24 bits left: FAINT in f32_rows.h).  An infinite x, or one that rounds to an infinite hi, has NaN among its
// terms, and every sum of products with it is NaN: the kernels do such rows over (f32_rows.h).
__device__ inline void split(float x, __bf16& hi, __bf16& mid, __bf16& lo) {
    hi = (__bf16)x;
    float r = x - (float)hi;
    mid = (__bf16)r;
    lo = (__bf16)(r - (float)mid);
}
// registers first .. first + 7 of a score tile as B operands
__device__ inline void split_regs(const f32x16& x, int first, bf16x8 (&o)[3]) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        __bf16 hi, mid, lo;
        split(x[first + e], hi, mid, lo);
        o[0][e] = hi; o[1][e] = mid; o[2][e] = lo;
    }
}
// Exponentials in base 2: log2(e) (and scale log2(e)) as hi + lo, so that the argument is formed
// with no more rounding than x * scale - m would have.
constexpr float L2E_HI = 1.44269502162933349609f, L2E_LO = 1.925963033500011079e-08f;
constexpr float LN2_HI = 0.693147182464599609375f, LN2_LO = -1.904654299957767878e-09f;
struct Scale2 {
    float hi, lo;
    __device__ explicit Scale2(float scale) {
        hi = scale * L2E_HI;
        lo = fmaf(scale, L2E_HI, -hi) + scale * L2E_LO;
    }
    // 2^(x (hi + lo) - m - m_lo); 0 for x = -inf (lo may be negative)
    __device__ float exp2(float x, float m, float m_lo) const {
        return __builtin_amdgcn_exp2f(fmaf(x, hi, -m) + fmaf(fmaxf(x, -1e30f), lo, -m_lo));
    }
};
// natural to base-2 units, as hi + lo.  x = +inf (no weight) is its hi; x = -inf and an x that
// overflows have a lo that makes the exponential NaN: see split.
__device__ inline void to_base2(float x, float& hi, float& lo) {
    hi = x * L2E_HI;
    lo = x == INFINITY ? 0.f : fmaf(x, L2E_HI, -hi) + x * L2E_LO;
}

}  // namespace sa
