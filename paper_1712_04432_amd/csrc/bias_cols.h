// Column sums of a bf16 Delta_Y with 16-byte row chunks (8 columns), shared by the column-sum
// kernel and the launches that carry them.
#pragma once

#include "common.h"

namespace imbd {

constexpr int BIAS_PITCH = 64 + 4;

// db[m] = alpha * sum_b dy[b][m] for the 64 columns from m_blk, by 256 threads (t: the index
// among them): thread t sums chunk t%8 over the rows r = t/8 + 32i in ascending order (eight
// loads in flight per batch), then the 32 row phases are added in phase order; optionally
// bias[m] -= lr * db[m]. M % 8 == 0. part: 32 rows of LDS. Every thread of the workgroup must
// call it (it holds a barrier).
__device__ __forceinline__ void bias_cols64(int M, int B, const uint16_t *__restrict__ dy, int64_t lddy, float alpha,
                                            float *__restrict__ db_out, float *__restrict__ bias, float lr, int m_blk,
                                            int t, float (*part)[BIAS_PITCH]) {
  const int j = t & 7, q = t >> 3;
  const int m0 = m_blk + 8 * j;
  const bool live = m0 < M;  // M % 8 == 0: a chunk is wholly in or out
  float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int r0 = q; r0 < B; r0 += 32 * 8) {
    u32x4 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int r = r0 + 32 * u;
      v[u] = live && r < B ? *reinterpret_cast<const u32x4 *>(dy + (int64_t)r * lddy + m0) : u32x4{0u, 0u, 0u, 0u};
    }
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        s[2 * e] += bf16_to_f32((uint16_t)(v[u][e] & 0xffffu));
        s[2 * e + 1] += bf16_to_f32((uint16_t)(v[u][e] >> 16));
      }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) part[q][8 * j + e] = s[e];
  __syncthreads();
  if (t < 64) {
    const int m = m_blk + t;
    float sum = 0.f;
    for (int k = 0; k < 32; ++k) sum += part[k][t];
    if (m < M) {
      const float g = alpha * sum;
      if (db_out) db_out[m] = g;
      if (bias) bias[m] = fmaf(-lr, g, bias[m]);
    }
  }
}

// Whether bias_cols64 takes the operand.
inline bool bias_cols64_ok(int M, const void *dy, int64_t lddy) {
  return M % 8 == 0 && lddy % 8 == 0 && (uintptr_t)dy % 16 == 0;
}

}  // namespace imbd
