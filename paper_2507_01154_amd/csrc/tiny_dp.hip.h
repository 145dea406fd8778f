// Algorithm 1 in one launch for fp32 layers of at most 64 x 64 and a few short samples: one workgroup, one wave per sample.
//
// Such a call is all launches and latency (32 x 32, B = 4, T = 16: contraction 5.0 us, clip factors 1.7, aggregation 3.2, and the gaps
// between them).  A wave forms its sample's gradient on v_mfma_f32_32x32x2 straight from memory - all loads of 16 tokens
// in flight at once, no staging -, takes its norm and factor, and leaves the gradient in LDS, where the workgroup then sums
// the samples in order and adds the noise as the streaming kernel would.  32 x 32, B = 4, T = 16, calls back to back, before and so, us:
// 10.2, 4.9 (the kernel 5.0).  One by one from Python, which takes 7 of them itself: 11.8, 7.5; B = 16: 14.3, 8.1; 64 x 64, B = 4, T = 16:
// 12.1, 7.8, T = 64: 17.6, 12.8; 30 x 34, B = 16, T = 64: 21.5, 20.1.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "elementwise.hip.h"
#include "gemm_mfma.hip.h"
#include "gemm_tile128.hip.h"

namespace flashdp {

struct TinyArgs {
  const float* X;        // [B][T][P]
  const float* dY;       // [B][T][D]
  int B, T, P, D;
  float* out_norms;      // [B] or nullptr
  float* out;            // [D][P]
  float C, noise_scale;
  uint64_t seed;
  uint32_t layer;
  int accumulate;
};
constexpr int TINY_SIDE = 64, TINY_TOKENS = 64, TINY_SAMPLES = 16, TINY_LDS_BYTES = 64 * 1024;

// FM x FN blocks of 32 x 32 cover D x P.
template <int FM, int FN>
__global__ __launch_bounds__(64 * TINY_SAMPLES) void tiny_dp_kernel(const TinyArgs a) {
  extern __shared__ __attribute__((aligned(16))) float G[];   // [B][D * P]
  __shared__ float fac[TINY_SAMPLES];
  const int lane = threadIdx.x & 63, i = threadIdx.x >> 6;    // sample
  const int half = lane >> 5, c = lane & 31, S = a.D * a.P;
  if (i < a.B) {   // waves beyond the samples only help with the sum
    const float* const y = a.dY + (size_t)i * a.T * a.D;
    const float* const x = a.X + (size_t)i * a.T * a.P;
    // An infinity meets the zeros beyond a ragged edge of the 64 x 64 tile that the other kernels use here, which makes
    // the sample's norm NaN: likewise.
    const bool ragged_d = a.D < TINY_SIDE, ragged_p = a.P < TINY_SIDE;
    float ragged = 0.0f;
    f32x16_t acc[FM][FN];
#pragma unroll
    for (int m = 0; m < FM; ++m)
#pragma unroll
      for (int n = 0; n < FN; ++n)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[m][n][e] = 0.0f;
#pragma unroll 1
    for (int t0 = 0; t0 < a.T; t0 += 16) {
      float fa[8][FM], fb[8][FN];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int t = t0 + 2 * k + half;
#pragma unroll
        for (int m = 0; m < FM; ++m) fa[k][m] = t < a.T && 32 * m + c < a.D ? y[t * a.D + 32 * m + c] : 0.0f;
#pragma unroll
        for (int n = 0; n < FN; ++n) fb[k][n] = t < a.T && 32 * n + c < a.P ? x[t * a.P + 32 * n + c] : 0.0f;
      }
#pragma unroll
      for (int k = 0; k < 8; ++k) {
#pragma unroll
        for (int m = 0; m < FM; ++m) ragged = fmaf(0.0f, ragged_p ? fa[k][m] : 0.0f, ragged);
#pragma unroll
        for (int n = 0; n < FN; ++n) ragged = fmaf(0.0f, ragged_d ? fb[k][n] : 0.0f, ragged);
      }
#pragma unroll
      for (int k = 0; k < 8; ++k)
#pragma unroll
        for (int m = 0; m < FM; ++m)
#pragma unroll
          for (int n = 0; n < FN; ++n) acc[m][n] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[k][m], fb[k][n], acc[m][n], 0, 0, 0);
    }
    // acc[m][n][4q + r] = element (32 m + 8 q + 4 half + r, 32 n + c), zero beyond D and P: a row's elements go to LDS side by side
    float ss[4] = {ragged, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int m = 0; m < FM; ++m)
#pragma unroll
      for (int n = 0; n < FN; ++n)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          ss[e & 3] = fmaf(acc[m][n][e], acc[m][n][e], ss[e & 3]);
          const int row = 32 * m + 8 * (e >> 2) + 4 * half + (e & 3), col = 32 * n + c;
          if (row < a.D && col < a.P) G[i * S + row * a.P + col] = acc[m][n][e];
        }
    const float w = wave_sum_to_lane63((ss[0] + ss[1]) + (ss[2] + ss[3]));
    if (lane == 63) {
      const double n = sqrt((double)w);
      fac[i] = clip_factor_of(n, a.C);
      if (a.out_norms) a.out_norms[i] = (float)n;
    }
  }
  // the noise of this thread's first group, and what the output holds, while the others get here
  const int groups = (S + 3) / 4;
  Normals4 z = {};
  if (a.noise_scale != 0.0f && (int)threadIdx.x < groups) z = noise_group(a.seed, a.layer, threadIdx.x);
  __syncthreads();
  for (int v = threadIdx.x; v < groups; v += blockDim.x) {
    float sum[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) sum[q] = a.accumulate && 4 * v + q < S ? a.out[4 * v + q] : 0.0f;
    for (int s = 0; s < a.B; ++s) {
      const float f = fac[s];
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (4 * v + q < S) sum[q] = fmaf(f, G[s * S + 4 * v + q], sum[q]);
    }
    if (a.noise_scale != 0.0f) {
      if (v != (int)threadIdx.x) z = noise_group(a.seed, a.layer, v);
#pragma unroll
      for (int q = 0; q < 4; ++q) sum[q] = fmaf(a.noise_scale, z.z[q], sum[q]);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (4 * v + q < S) a.out[4 * v + q] = sum[q];
  }
}

}  // namespace flashdp
