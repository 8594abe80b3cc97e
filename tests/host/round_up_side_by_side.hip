// Blocks that change the rounding mode, with nothing between them: looked at as assembly, never run.
#include "lq_round_up.h"

__global__ void side_by_side(const float* in, uint32_t* out, float* four) {
  const int i = threadIdx.x;
  const float z = in[i], s = in[i + 64], k = in[i + 128];
  float a[4] = {z, s, k, z}, b[4] = {s, k, z, k};
  uint32_t f[8];
  __builtin_amdgcn_sched_barrier(0);
  lq::sum_up(z, s, k, s, z, k, f + 0, f + 1);
  lq::sum_up(k, s, z, s, k, z, f + 2, f + 3);
  lq::sum_up_f16(z, s, k, s, z, k, f + 4, f + 5);
  lq::sum_up_f16(k, s, z, s, k, z, f + 6, f + 7);
  lq::fma_up(a, s, z);
  lq::fma_up(b, k, s);
  __builtin_amdgcn_sched_barrier(0);
  for (int j = 0; j < 8; ++j) out[8 * i + j] = f[j];
  for (int j = 0; j < 4; ++j) four[8 * i + j] = a[j], four[8 * i + 4 + j] = b[j];
}
