// The bf16 matrix instruction with its accumulators in AGPRs, written out as instructions.
#pragma once
#include <hip/hip_runtime.h>

namespace emoe {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

// Reads one accumulator where it lives (an AGPR).  Written out as an instruction so that the compiler
// moves accumulators to VALU registers one at a time, where they are used, instead of copying all
// 256 of them out at the end of the K loop (which needs every VGPR and spills the rest).
__device__ __forceinline__ float acc_read(float a) {
    float v;
    asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v) : "a"(a));
    return v;
}

// The matrix instruction, written out with its accumulator tied to AGPRs: with 64 accumulators of four registers filling
// all 256 AGPRs the compiler's own allocation moves them between AGPRs and VGPRs inside the loop (500 moves per K tile).
// The compiler does not see matrix instructions in these statements and adds none of the wait states they need, so
//  - operands come from LDS reads (waited for by counter) and accumulators from other matrix instructions (mfma_16x16x32_first, mfma_zero);
//  - mfma_zero, whose operand is a constant that the compiler writes wherever it likes, also between two of these
//    statements, brings along the two wait states that a VALU write of an operand needs;
//  - mfma_settle(), more wait states than the longest the ISA asks for, stands between the last one and the first read
//    of an accumulator, and between the last read and the next item's first one.
__device__ __forceinline__ void mfma_16x16x32(floatx4& acc, const bf16x8& w, const bf16x8& x) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(w), "v"(x));
}
// the first one of an accumulator: nothing to add to (with wait states of its own, as mfma_zero; they pass while the one before runs)
__device__ __forceinline__ void mfma_16x16x32_first(floatx4& acc, const bf16x8& w, const bf16x8& x) {
    asm volatile("s_nop 1\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=a"(acc) : "v"(w), "v"(x));
}
__device__ __forceinline__ void mfma_zero(floatx4& acc, const bf16x8& zero) {  // 0 * 0 + 0
    asm volatile("s_nop 1\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %1, 0" : "=a"(acc) : "v"(zero));
}
__device__ __forceinline__ void mfma_settle() { asm volatile("s_nop 15\n\ts_nop 15" ::: "memory"); }

}  // namespace
}  // namespace emoe
