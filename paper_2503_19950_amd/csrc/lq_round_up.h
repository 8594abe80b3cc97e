// Sums and conversions rounded towards +infinity.  The wavefront's rounding mode changes inside one asm block and is back to
// nearest at its end, so that no other instruction can run under it.  Two writes of the mode register need two instructions
// between them: two blocks may be placed side by side, and the compiler, which would see to that for its own writes, does
// not look into asm.  So every block begins with the wait.  (No other instruction of these kernels writes or reads the mode.)
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lq {

#define LQ_ROUND_UP "s_nop 1\n\ts_setreg_imm32_b32 hwreg(HW_REG_MODE, 0, 4), 5\n\t"   // fp32 and fp16/fp64
#define LQ_ROUND_NEAREST "s_setreg_imm32_b32 hwreg(HW_REG_MODE, 0, 4), 0"

// bits of z0 + k0 s0 and z1 + k1 s1 rounded up to fp32
__device__ __forceinline__ void sum_up(float z0, float s0, float k0, float z1, float s1, float k1, uint32_t* f0, uint32_t* f1) {
  asm(LQ_ROUND_UP
      "v_fma_f32 %0, %2, %3, %4\n\t"
      "v_fma_f32 %1, %5, %6, %7\n\t"
      LQ_ROUND_NEAREST
      : "=&v"(*f0), "=&v"(*f1) : "v"(k0), "v"(s0), "v"(z0), "v"(k1), "v"(s1), "v"(z1));
}
// the same, rounded up once more to fp16
__device__ __forceinline__ void sum_up_f16(float z0, float s0, float k0, float z1, float s1, float k1, uint32_t* f0, uint32_t* f1) {
  asm(LQ_ROUND_UP
      "v_fma_f32 %0, %2, %3, %4\n\t"
      "v_fma_f32 %1, %5, %6, %7\n\t"
      "v_cvt_f16_f32 %0, %0\n\t"
      "v_cvt_f16_f32 %1, %1\n\t"
      LQ_ROUND_NEAREST
      : "=&v"(*f0), "=&v"(*f1) : "v"(k0), "v"(s0), "v"(z0), "v"(k1), "v"(s1), "v"(z1));
}
// t[i] = z + t[i] s rounded up to fp32
__device__ __forceinline__ void fma_up(float (&t)[4], float s, float z) {
  asm(LQ_ROUND_UP
      "v_fma_f32 %0, %0, %4, %5\n\t"
      "v_fma_f32 %1, %1, %4, %5\n\t"
      "v_fma_f32 %2, %2, %4, %5\n\t"
      "v_fma_f32 %3, %3, %4, %5\n\t"
      LQ_ROUND_NEAREST
      : "+&v"(t[0]), "+&v"(t[1]), "+&v"(t[2]), "+&v"(t[3]) : "v"(s), "v"(z));
}

#undef LQ_ROUND_UP
#undef LQ_ROUND_NEAREST

}  // namespace lq
