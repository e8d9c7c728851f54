// Accumulation registers of a wavefront by number.
//
// As variables of the compiler, tied to that file or not, long-lived accumulators were carried to vector registers and
// scratch memory and back around every loop (444 spilled registers in the dK/dV kernel above 128 columns).  Each statement
// declares the whole file as overwritten, so that nothing of the compiler's lives there across one; it has no reason to
// use the file at all while its own values fit the 256 vector registers.  The build looks that outside of these statements
// no instruction of such a kernel names one, and for the wait states of all products in asm statements (asm_check.py).
#pragma once
#include "mfma_tiles.h"

namespace sa {

#ifdef __HIP_DEVICE_COMPILE__
#define ACC_TEN(b) "a" #b "0", "a" #b "1", "a" #b "2", "a" #b "3", "a" #b "4", "a" #b "5", "a" #b "6", "a" #b "7", "a" #b "8", "a" #b "9"
#define ACC_FILE                                                                                                   \
    "a0", "a1", "a2", "a3", "a4", "a5", "a6", "a7", "a8", "a9", ACC_TEN(1), ACC_TEN(2), ACC_TEN(3), ACC_TEN(4), ACC_TEN(5),    \
        ACC_TEN(6), ACC_TEN(7), ACC_TEN(8), ACC_TEN(9), ACC_TEN(10), ACC_TEN(11), ACC_TEN(12), ACC_TEN(13), ACC_TEN(14), ACC_TEN(15), \
        ACC_TEN(16), ACC_TEN(17), ACC_TEN(18), ACC_TEN(19), ACC_TEN(20), ACC_TEN(21), ACC_TEN(22), ACC_TEN(23), ACC_TEN(24),        \
        "a250", "a251", "a252", "a253", "a254", "a255"
#else
#define ACC_FILE        // the host pass knows none of these names
#endif
__device__ __forceinline__ void acc_zero(int i) { asm volatile("v_accvgpr_write_b32 a[%0], 0" : : "n"(i) : ACC_FILE); }
__device__ __forceinline__ void acc_write(int i, float x) { asm volatile("v_accvgpr_write_b32 a[%0], %1" : : "n"(i), "v"(x) : ACC_FILE); }
__device__ __forceinline__ float acc_read(int i) {
    float x;
    asm volatile("v_accvgpr_read_b32 %0, a[%1]" : "=v"(x) : "n"(i) : ACC_FILE);
    return x;
}
// block += a b.  The two wait states stand in every one: b is packed by vector instructions, which the
// compiler moves up to the very product that reads it, and its hazard recogniser does not see this one
// (without them single columns of dK were wrong now and then).  They pass while the product before runs.
__device__ __forceinline__ void acc_mfma(int block, bf16x8 a, bf16x8 b) {
    asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 a[%2:%3], %0, %1, a[%2:%3]"
                 : : "v"(a), "v"(b), "n"(16 * block), "n"(16 * block + 15) : ACC_FILE);
}
// without the wait: where the vector instructions that pack b lie further back, behind other products (the build
// looks for that in the assembly)
__device__ __forceinline__ void acc_mfma_far(int block, bf16x8 a, bf16x8 b) {
    asm volatile("v_mfma_f32_32x32x16_bf16 a[%2:%3], %0, %1, a[%2:%3]"
                 : : "v"(a), "v"(b), "n"(16 * block), "n"(16 * block + 15) : ACC_FILE);
}
// The last products before their results are read.
__device__ __forceinline__ void acc_settle() { asm volatile("s_nop 15\n\ts_nop 15" : : : ACC_FILE); }

}  // namespace sa
