// Algorithm 1 for rows without a sequence (T = 1).  A per-sample gradient is then the outer product G_i = dy_i x_i^T and
// its squared norm is |dy_i|^2 |x_i|^2 exactly: sums of squares, without the cancellation that the Gram form of longer
// sequences has.  So nothing of size B * D * P is computed twice or parked: one kernel takes the norms and clip factors
// from the rows, a second one forms sum_i (c_i dy_i) x_i^T as a plain product over the batch, with the noise in its
// epilogue.  Everything is fp32 (norms fp64) for every storage type.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "edge_plan.h"
#include "elementwise.hip.h"
#include "gemm_mfma.hip.h"
#include "gemm_simple.hip.h"

namespace flashdp {

struct RowsArgs {
  const void* X;         // [B][P]
  const void* dY;        // [B][D]
  int B, P, D;
  int tiles_m, tiles_n;
  float* factors;        // [B]
  float* out_norms;      // [B] or nullptr
  float* out;            // [D][P]
  float C, noise_scale;
  uint64_t seed;
  uint32_t layer;
  int accumulate;
};

// 16 bytes from element e on (any element: rows need not be aligned to more than their type) as fp32.
template <int DT>
__device__ __forceinline__ void rows_load16b(const void* p, size_t e, float* f) {
  if constexpr (DT == DT_F32) {
    const f32x4_any_t v = *(const f32x4_any_t*)((const float*)p + e);
    f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
  } else {
    widen8<DT>(*(const u32x4_any_t*)((const unsigned short*)p + e), f);
  }
}

// This thread's share of a row's sum of squares, V elements (1, or 16 bytes of them) per load.
template <int DT, int V>
__device__ __forceinline__ double row_square_sum_v(const void* p, size_t base, int n) {
  constexpr int Q = edge_plan::WALK_CHUNKS;
  double s[4] = {0.0, 0.0, 0.0, 0.0};
  edge_plan::walk_row<V>(n, threadIdx.x, [&](uint32_t k) {
    float v[Q][V];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const uint32_t kq = k + 256 * V * q;
      if (V > 1 && kq + V <= (uint32_t)n) {
        if constexpr (V > 1) rows_load16b<DT>(p, base + kq, v[q]);
      } else {
#pragma unroll
        for (int e = 0; e < V; ++e) v[q][e] = kq + e < (uint32_t)n ? load_elem<DT>(p, base + kq + e) : 0.0f;
      }
    }
#pragma unroll
    for (int q = 0; q < Q; ++q)
#pragma unroll
      for (int e = 0; e < V; ++e) s[(q + e) & 3] = fma((double)v[q][e], (double)v[q][e], s[(q + e) & 3]);
  });
  return (s[0] + s[1]) + (s[2] + s[3]);
}

// Sum of squares of one row by a workgroup's 256 threads (this thread's share).  One workgroup reads the whole row and
// is bound by the latency of its loads, so every thread has four in flight: of one element where two steps of those
// take the row (16-bit, B = 17, 301 x 70: 13.1 us a call, 14.4 with 16-byte loads on a tenth of the threads), of 16
// bytes for longer ones (fp32, B = 2, 200000 x 8: 88 us with elements, 51; bf16, 13824 x 64: 14.3, 11.9).
template <int DT>
__device__ __forceinline__ double row_square_sum(const void* p, size_t base, int n) {
  if (n <= 2048) return row_square_sum_v<DT, 1>(p, base, n);
  return row_square_sum_v<DT, DT == DT_F32 ? 4 : 8>(p, base, n);
}

// n_i and c_i, one workgroup per sample.
template <int DT>
__global__ __launch_bounds__(256) void rows_clip_kernel(const RowsArgs a) {
  __shared__ double red[8];
  const int i = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double sx = row_square_sum<DT>(a.X, (size_t)i * a.P, a.P);
  double sy = row_square_sum<DT>(a.dY, (size_t)i * a.D, a.D);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    sx += __shfl_xor(sx, off, 64);
    sy += __shfl_xor(sy, off, 64);
  }
  if (lane == 0) { red[wave] = sx; red[4 + wave] = sy; }
  __syncthreads();
  if (threadIdx.x == 0) {
    const double n = sqrt(((red[0] + red[1]) + (red[2] + red[3])) * ((red[4] + red[5]) + (red[6] + red[7])));
    // G_i is never formed, so its overflow has to be brought in here: where n_i is no fp32 number the factor is NaN and
    // poisons out_grad (C / n_i would underflow to a finite zero and drop the sample in silence).
    const float nf = (float)n;
    a.factors[i] = __builtin_isinf(nf) ? __builtin_nanf("") : clip_factor_of(n, a.C);
    if (a.out_norms) a.out_norms[i] = nf;
  }
}

// Four consecutive elements (cols col..col+3 of row `row`) as fp32; elements past n and rows past rows are zero.
template <int DT>
__device__ __forceinline__ f32x4_any_t rows_load4(const void* p, int row, int rows, int col, int n, bool vec) {
  f32x4_any_t v = {0.0f, 0.0f, 0.0f, 0.0f};
  if (row >= rows || col >= n) return v;
  const size_t e = (size_t)row * n + col;
  if (vec) {   // n % 4 == 0: the group is all in, and aligned like its operand (16 bytes) to four elements
    if constexpr (DT == DT_F32) {
      const float4 f = *(const float4*)((const float*)p + e);
      v = f32x4_any_t{f.x, f.y, f.z, f.w};
    } else {
      const uint2 u = *(const uint2*)((const unsigned short*)p + e);
      float f[8];
      widen8<DT>(u32x4_t{u.x, u.y, 0, 0}, f);
      v = f32x4_any_t{f[0], f[1], f[2], f[3]};
    }
  } else {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (col + q < n) v[q] = load_elem<DT>(p, e + q);
  }
  return v;
}

// Bound by latency where the batch is long and the tiles few (256 x 784 x 512: 13 x 8 workgroups, one reduction of 256
// rows each), hence 64-wide tiles there, and by the write of the output with its noise where the layer is large.
// Both kernels together, one call, fp32, against parking the per-sample gradients: B = 256, 784 x 512: 17 us, 250 before;
// B = 16, 4096 x 4096: 49, 703; B = 1, 768 x 3072: 15, 28.  bf16: 22, 127; 43, 260; two
// samples, 4096 x 13824: 125, 163.
// out = (accumulate ? out : 0) + sum_i (c_i dy_i) x_i^T + noise on v_mfma_f32_32x32x2_f32.  4 waves, each F x F blocks of
// 32 x 32; two LDS stages as in the fp32 per-sample kernel (operands as in memory, pitch 32 floats mod 64, the next
// rows fetched into registers meanwhile).  The clip factor is multiplied in while dY is staged.
template <int F>
struct RowsCfg {
  static constexpr int BM = 64 * F, BK = 32 / F;           // tile side; rows (samples) per step
  static constexpr int LD = BM + 32;                       // 96 resp. 160 floats: 32 mod 64
  static constexpr int CPR = BM / 4, RSTEP = 256 / CPR;    // 16-byte chunks per row; rows per pass
  static_assert(BK == 2 * RSTEP, "two chunks per thread and operand");
};

template <int F, int DT>
__global__ __launch_bounds__(256) void rows_accum_kernel(const RowsArgs a) {
  using Cfg = RowsCfg<F>;
  constexpr int BK = Cfg::BK, LD = Cfg::LD;
  constexpr int STAGE = BK * LD;
  __shared__ __attribute__((aligned(16))) float lds[4 * STAGE];   // two stages of dY rows, two of X rows; output rows at the end
  float* const As = lds;
  float* const Bs = lds + 2 * STAGE;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int tm, tn;
  tile_coords<8>(xcd_remap(blockIdx.x, a.tiles_m * a.tiles_n), a.tiles_m, a.tiles_n, &tm, &tn);
  const int m0 = tm * Cfg::BM, n0 = tn * Cfg::BM;
  const int c_row = tid / Cfg::CPR, c_col = (tid % Cfg::CPR) * 4;
  const bool avec = a.D % 4 == 0, bvec = a.P % 4 == 0;

  f32x4_any_t ra[2], rb[2];
  float rc[2];
  auto fetch = [&](int s0) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int s = s0 + c_row + j * Cfg::RSTEP;
      ra[j] = rows_load4<DT>(a.dY, s, a.B, m0 + c_col, a.D, avec);
      rb[j] = rows_load4<DT>(a.X, s, a.B, n0 + c_col, a.P, bvec);
      rc[j] = s < a.B ? a.factors[s] : 0.0f;
    }
  };
  auto stage = [&](int st) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int o = (c_row + j * Cfg::RSTEP) * LD + c_col;
      *(float4*)(As + st * STAGE + o) = make_float4(rc[j] * ra[j].x, rc[j] * ra[j].y, rc[j] * ra[j].z, rc[j] * ra[j].w);
      *(float4*)(Bs + st * STAGE + o) = make_float4(rb[j].x, rb[j].y, rb[j].z, rb[j].w);
    }
  };

  f32x16_t acc[F][F];
#pragma unroll
  for (int i = 0; i < F; ++i)
#pragma unroll
    for (int j = 0; j < F; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

  const int wm = (wave & 1) * 32 * F, wn = (wave >> 1) * 32 * F;
  const int fr = (lane >> 5) * LD + (lane & 31);
  const int nk = (a.B + BK - 1) / BK;
  fetch(0);
  stage(0);
  for (int k = 0; k < nk; ++k) {
    const int cur = k & 1;
    fetch((k + 1) * BK);   // past the last row: zeros, nothing is read
    __syncthreads();       // step k is staged; everyone is done with the other stage
#pragma unroll
    for (int ks = 0; ks < BK / 2; ++ks) {
      float fa[F], fb[F];
#pragma unroll
      for (int i = 0; i < F; ++i) {
        fa[i] = As[cur * STAGE + fr + 2 * ks * LD + wm + 32 * i];
        fb[i] = Bs[cur * STAGE + fr + 2 * ks * LD + wn + 32 * i];
      }
#pragma unroll
      for (int i = 0; i < F; ++i)
#pragma unroll
        for (int j = 0; j < F; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fb[j], fa[i], acc[i][j], 0, 0, 0);
    }
    stage(cur ^ 1);
  }

  // acc[i][j][4q + r] = element (m0 + wm + 32i + lane % 32, n0 + wn + 32j + 8q + 4 (lane / 32) + r).  64 rows at a time go
  // through LDS, so that whole rows are written and the noise generator stands in one rolled loop.
  constexpr int OP = Cfg::BM + 4;
  static_assert(64 * OP <= 4 * STAGE, "output rows fit the stages");
#pragma unroll
  for (int i = 0; i < F; ++i) {
    __syncthreads();
#pragma unroll
    for (int j = 0; j < F; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *(float4*)(lds + ((wave & 1) * 32 + (lane & 31)) * OP + wn + 32 * j + 8 * q + 4 * (lane >> 5)) =
            make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
    __syncthreads();
    // A thread takes groups of four elements of the output that share a noise group, whatever the row's first element is:
    // with P no multiple of 4 the first and the last group of a tile's row may be partly another tile's.  (Groups of four
    // columns instead draw two noise groups each and store element by element: bf16, B = 2, 70 x 1820: 21 us a call, 16; 4001 x 5001: 80, 56.)
    const int gpr = bvec ? Cfg::CPR : Cfg::CPR + 1;   // groups that a tile's row touches
#pragma unroll 1
    for (int c = tid; c < 64 * gpr; c += 256) {
      const int r64 = bvec ? c / Cfg::CPR : c / (Cfg::CPR + 1);
      const int row = m0 + (r64 >> 5) * 32 * F + 32 * i + (r64 & 31);
      if (row >= a.D) continue;
      const size_t e_tile = (size_t)row * a.P + n0;             // the row's first element in this tile
      const int cc = (c - r64 * gpr) * 4 - (int)(e_tile & 3);   // the group's first column in the tile
      const int lo = max(0, -cc), hi = min(4, min(Cfg::BM, a.P - n0) - cc);
      if (hi <= lo) continue;
      float v[4];
      if (bvec) {
        const float4 t = *(const float4*)(lds + r64 * OP + cc);
        v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = lds[r64 * OP + min(max(cc + r, 0), Cfg::BM - 1)];
      }
      const size_t e = e_tile + cc;
      if (a.noise_scale != 0.0f) {
        const Normals4 z = noise_group(a.seed, a.layer, e >> 2);
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = fmaf(a.noise_scale, z.z[r], v[r]);
      }
      float* po = a.out + e;
      if (lo == 0 && hi == 4 && !a.accumulate) {
        typedef float f32x4_t __attribute__((ext_vector_type(4)));
        __builtin_nontemporal_store((f32x4_t){v[0], v[1], v[2], v[3]}, (f32x4_t*)po);
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (r >= lo && r < hi) po[r] = a.accumulate ? po[r] + v[r] : v[r];
      }
    }
  }
}

}  // namespace flashdp
