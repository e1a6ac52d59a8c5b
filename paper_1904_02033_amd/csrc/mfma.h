// Matrix products of two shapes in one sum.
#pragma once
#include <hip/hip_runtime.h>

namespace sanns {

// Between matrix products of one shape and products of another that add to
// their sums.  A product takes the sum of one of its own shape straight from the
// pipeline; of another shape it reads the registers, five wait states after the
// product that writes them was issued at the earliest, and the hardware does not
// hold it back.  AMD clang 22 (ROCm 7.2) inserts no wait for it: with
// v_mfma_i32_16x16x32_i8 less than five wait states behind the
// v_mfma_i32_16x16x64_i8 whose sum it adds to (four the other way round), half of
// the four registers of every lane came out wrong, every time.  The scheduling
// barriers keep all products of the first shape before the wait and all of the
// second behind it, so the distance does not hang on the compiler's order.
__device__ __forceinline__ void mfma_shape_change() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_nop 7");
  __builtin_amdgcn_sched_barrier(0);
}

}  // namespace sanns
