// Matrix instructions on accumulators that stay in their accumulation registers.  With all of them there and the fragments of two
// steps in vector registers, the compiler's own form (result and addend in different registers) left 80 - 170 register copies per 128
// instructions of the GEMM kernels; and with the attention's scores in vector registers it keeps the other accumulators there too.
//
// The compiler sees neither these instructions nor their latency:
//   * operands that vector instructions write have to be there two wait states earlier (an empty statement that names the finished
//     operand, ahead of some other instruction, keeps its last write from sinking to the use);
//   * whoever reads the accumulators calls mfma_drain first.  A wait alone holds nothing back: reads of registers are not memory, and
//     the scheduler took those of dK and dV above it.  (Naming the accumulators in a statement behind the wait is no fence either: the
//     register allocator then copied 128 of them ahead of it, at the end of the dK/dV kernel's loop.)
// The compiler may still copy or spill an accumulator where it likes: tests/test_mfma_in_place.py reads from the compiled code
// that none is touched ahead of the wait, that the operands are there in time, and that nothing is spilled.
#pragma once
#include "common.h"

namespace beagle {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 mfma_bf16x8_t;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float mfma_f32x16_t;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float mfma_f32x4_t;

// 16 x 16 (four values per lane) and 32 x 32 (sixteen) accumulators
__device__ __forceinline__ void mfma_in_place(mfma_f32x4_t& acc, const mfma_bf16x8_t& a, const mfma_bf16x8_t& b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}
__device__ __forceinline__ void mfma_in_place(mfma_f32x16_t& acc, const mfma_bf16x8_t& a, const mfma_bf16x8_t& b) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}

// the results of every instruction issued so far are in their accumulators, and nothing that reads those moves up
__device__ __forceinline__ void mfma_drain() {
  asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

}  // namespace beagle
