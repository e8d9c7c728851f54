// What the three-term kernels (f32x3_step.hip, f32x3_split.hip) share: terms made in steps that go beside products, and
// the six products of two three-term operands.
#pragma once
#include "mfma_tiles.h"

namespace sa {

typedef bf16x8 bf16x8x3[3];

// Eight numbers as three terms each: 11 vector instructions a pair, in six steps that go beside one product each.
// (What a term leaves as a dot product with (-1, 0), one instruction instead of two, is no gain: the matrix core
// does not work beside those.)
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
struct Split8 {
    float x[8], y[8];           // what is left, the last term
    bf16x2 t[3][4];
    template <int P>
    __device__ __forceinline__ void round() {
        typedef float f32x2 __attribute__((ext_vector_type(2)));
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const f32x2 v = {x[2 * i], x[2 * i + 1]};
            t[P][i] = __builtin_convertvector(v, bf16x2);
        }
    }
    template <int P>
    __device__ __forceinline__ void widen(int first, int end) {
#pragma unroll
        for (int i = first; i < end; ++i) {
            const uint32_t w = __builtin_bit_cast(uint32_t, t[P][i]);
            y[2 * i] = __uint_as_float(w << 16);
            y[2 * i + 1] = __uint_as_float(w & 0xffff0000u);
        }
    }
    __device__ __forceinline__ void rest(int first, int end) {
#pragma unroll
        for (int i = 2 * first; i < 2 * end; ++i) x[i] -= y[i];
    }
    __device__ __forceinline__ void step(int i) {
        if (i == 0) { round<0>(); widen<0>(0, 2); }
        if (i == 1) { widen<0>(2, 4); rest(0, 2); }
        if (i == 2) { rest(2, 4); round<1>(); }
        if (i == 3) widen<1>(0, 4);
        if (i == 4) rest(0, 4);
        if (i == 5) round<2>();
    }
    __device__ __forceinline__ void operands(bf16x8 (&o)[3]) const {
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            struct Quad { bf16x2 t[4]; } q = {t[p][0], t[p][1], t[p][2], t[p][3]};
            o[p] = __builtin_bit_cast(bf16x8, q);
        }
    }
};
__device__ __forceinline__ void split8(const float (&x)[8], bf16x8 (&o)[3]) {
    Split8 c;
#pragma unroll
    for (int e = 0; e < 8; ++e) c.x[e] = x[e];
#pragma unroll
    for (int i = 0; i < 6; ++i) c.step(i);
    c.operands(o);
}
// registers first .. first + 7 of a score tile
__device__ inline void split_tile(const f32x16& w, int first, bf16x8 (&o)[3]) {
    float x[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = w[first + e];
    split8(x, o);
}
// The six products of a b, smallest first but for the leading one in their midst: hi += that, lo += the others.
// beside(i) goes with the i-th.
constexpr int LEADING = 2, TERM_A[6] = {1, 2, 0, 0, 1, 0}, TERM_B[6] = {1, 0, 0, 2, 0, 1};
template <typename Beside>
__device__ __forceinline__ void products(const bf16x8 (&a)[3], const bf16x8 (&b)[3], f32x16& hi, f32x16& lo, Beside beside) {
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        __builtin_amdgcn_sched_barrier(0);
        f32x16& c = i == LEADING ? hi : lo;
        c = mfma(a[TERM_A[i]], b[TERM_B[i]], c);
        __builtin_amdgcn_sched_barrier(0);
        beside(i);
    }
}
}  // namespace sa
