// The parking pass for fp32 inputs on the bfloat16 matrix cores: every operand element is split into three bfloat16 parts that
// add up to it exactly, x = x1 + x2 + x3 (8 + 8 + 8 significant bits, each part the rounding of what the ones before leave;
// the technique of Henry, Tang and Heinecke, "Leveraging the bfloat16 artificial intelligence datatype for higher-precision
// computations", 2019), and a product is formed of all pairs of parts but x3 y3, which is below 2^-33 of it.
//
// Why.  Bound by the fp32 matrix rate (157 TFLOP/s) before; eight bfloat16 products on a sixteen times faster unit.  A wave
// issues eight times 16 matrix instructions a k-tile, so the splitting (about 9 vector instructions an element) runs beside the other
// workgroup's products.  128 x 128 tiles, 4 waves of 64 x 64, one 48 KB LDS stage (3 parts x 2 operands x 32 rows of 128),
// the next k-tile in registers meanwhile, two workgroups per CU.
//
// The products x1 y1 have an accumulator of their own, the seven smaller ones share another, and the two are added at the
// end.  So the large accumulator is rounded once in 32 tokens (matrix instructions do not round an addition as carefully as
// an fp32 one), the other's roundings are 2^-8 of that, and a product that stands alone is rounded once.  Relative error of a
// gradient against fp64 (2-norm), on the fp32 matrix instructions, with six products in one accumulator, and so: normal data, T = 2048:
// 8.1e-7, 7.0e-7, 2.7e-7; T = 333: 3.3e-7, 2.7e-7, 1.0e-7; T = 16: 7.4e-8, 3.4e-8, 3.2e-8; one token alone: 2.54e-8, 3.4e-8, 2.54e-8
// (largest element 5.96e-8, 1.5e-7, 5.97e-8); one token a thousand times the others, T = 2048: 8.1e-7, 5.1e-7, 2.9e-7; T = 16: 7.2e-8,
// 5.0e-8, 5.6e-8; T = 8: 5.1e-8, 5.1e-8, 5.4e-8; T = 4: 3.6e-8, 4.2e-8, 4.5e-8: below 16 tokens the fp32 instructions keep the layer.
// Larger than theirs, at about one rounding of fp32: a dominating token that comes last (products a hundred times the others' and more, any T: 2.5e-8,
// 4.5e-8 to 6.4e-8; they round it once, a matrix instruction of 32 tokens cuts the small products off beside it), and softmax-shaped values
// in both operands up to T = 33 (T = 16: 3.9e-8, 5.5e-8; T = 33: 6.4e-8, 6.6e-8; T = 100: 1.14e-7, 8.9e-8).
//
// fp32, contraction in us, on the fp32 matrix instructions and so: 4096 x 4096, B = 4, T = 2048: 2163, 1621 (170 TFLOP/s; six products 1402);
// 768 x 3072, B = 4, T = 1024: 248, 166; 64 x 448, B = 14, T = 1024: 237, 65; 128 x 13184, B = 1, T = 276: 76, 24; 1028 x 764, B = 8, T = 333:
// 93, 44.  The large ones are limited by power: a first call after a pause takes 1.7 to 2.0 ms where calls in a row take 1.6.
//
// Operands are scaled by 2^24 on their way into the parts and the sums by 2^-48 on their way out, both exact, so that the last part
// of the smallest float is a normal number and no product of parts is subnormal unless the product itself vanishes.
//
// What that does not cover is left to a plain fp32 loop over the tile, decided per workgroup: sums that are not finite (an infinity
// times a part that is zero or of the other sign is NaN) or whose squares overflow, operands from 2^103 and sums from 2^80 up.  Such a
// tile takes six to seven times as long: 4096 x 4096, B = 4, T = 2048, an infinity in every tile: 10.4 ms a call, 1.7 otherwise (one
// value of 1e-34 in every tile, which this loop used to redo: 10.2, 1.7).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gemm_mfma.hip.h"
#include "gemm_tile128.hip.h"
#include "tile128_plan.h"

namespace flashdp {

struct F32x3Cfg {
  static constexpr int NT = 256;
  static constexpr int PART = tile128_plan::OPERAND_ELEMS;        // elements of one part of one operand tile
  static constexpr int LDS_BYTES = 6 * PART * 2;                  // 48 KB
  static constexpr int OUT_PITCH = 128 + 4;
  static constexpr float SCALE = 0x1p24f, UNSCALE = 0x1p-48f;     // of operands; of sums of products
  static_assert(64 * OUT_PITCH * 4 <= LDS_BYTES, "output rows fit the stage");
};

// The three parts of two floats times 2^24 (low half: a).
__device__ __forceinline__ void split3(float a, float b, uint32_t* parts) {
  a *= F32x3Cfg::SCALE;
  b *= F32x3Cfg::SCALE;
  const uint32_t p1 = pack2_16bit<DT_BF16>(a, b);
  const float ra = a - __builtin_bit_cast(float, p1 << 16), rb = b - __builtin_bit_cast(float, p1 & 0xFFFF0000u);
  const uint32_t p2 = pack2_16bit<DT_BF16>(ra, rb);
  const float sa = ra - __builtin_bit_cast(float, p2 << 16), sb = rb - __builtin_bit_cast(float, p2 & 0xFFFF0000u);
  parts[0] = p1;
  parts[1] = p2;
  parts[2] = pack2_16bit<DT_BF16>(sa, sb);
}

// a.scratch: [B][D][P] fp32; a.partials: [B][tiles]; a.splits == B (one workgroup per tile and sample).
__global__ __launch_bounds__(256, 2) void gemm_f32x3_kernel(const Tile128Layer a) {
  namespace tp = tile128_plan;
  constexpr int PART = F32x3Cfg::PART;
  extern __shared__ __attribute__((aligned(16))) unsigned short lds[];   // parts 1..3 of the dY tile, then of the X tile
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wave_m = wave & 1, wave_n = wave >> 1;

  const int tiles = a.tiles_m * a.tiles_n, total = tiles * a.splits;
  if ((int)blockIdx.x >= total) return;   // the whole workgroup, before any barrier
  const int item = xcd_remap(blockIdx.x, total);
  const int sample = item / tiles, tile = item - sample * tiles;
  int tm, tn;
  tile_coords<8>(tile, a.tiles_m, a.tiles_n, &tm, &tn);
  const int m0 = tm * tp::SIDE, n0 = tn * tp::SIDE;
  const int T = a.T, P = a.P, D = a.D;

  // ---- global -> registers: 8 columns (two 16-byte loads) of rows r0 and r0 + 16 of either operand; what lies outside reads 0
  const int r0 = tid >> 4, c0 = 8 * (tid & 15);
  const uint32_t a_bytes = (uint32_t)T * (uint32_t)D * 4u, b_bytes = (uint32_t)T * (uint32_t)P * 4u;
  const char* const pa = (const char*)a.dY + (size_t)sample * a_bytes;
  const char* const pb = (const char*)a.X + (size_t)sample * b_bytes;
  const __amdgpu_buffer_rsrc_t rsa = make_rsrc(pa, a_bytes), rsb = make_rsrc(pb, b_bytes);
  uint32_t a_off[2], b_off[2];   // of the two loads; D and P are multiples of 4: a load is all in or all out
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    a_off[h] = m0 + c0 + 4 * h < D ? (uint32_t)(r0 * D + m0 + c0 + 4 * h) * 4u : 0x80000000u;
    b_off[h] = n0 + c0 + 4 * h < P ? (uint32_t)(r0 * P + n0 + c0 + 4 * h) * 4u : 0x80000000u;
  }
  const uint32_t a_half = 16u * (uint32_t)D * 4u, b_half = 16u * (uint32_t)P * 4u;
  u32x4_t raw_a[4], raw_b[4];
  auto fetch = [&]() {   // and move on by a k-tile; rows >= T read as zeros
#pragma unroll
    for (int q = 0; q < 4; ++q) raw_a[q] = __builtin_amdgcn_raw_buffer_load_b128(rsa, (int)(a_off[q & 1] + (q >> 1) * a_half), 0, 0);
#pragma unroll
    for (int q = 0; q < 4; ++q) raw_b[q] = __builtin_amdgcn_raw_buffer_load_b128(rsb, (int)(b_off[q & 1] + (q >> 1) * b_half), 0, 0);
#pragma unroll
    for (int h = 0; h < 2; ++h) { a_off[h] += 2 * a_half; b_off[h] += 2 * b_half; }
  };
  const int w_off = tp::kept_at(r0, c0);   // rows + 16 keep the swizzle
  auto stage = [&]() {
#pragma unroll
    for (int op = 0; op < 2; ++op)
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const u32x4_t lo = op == 0 ? raw_a[2 * q] : raw_b[2 * q], hi = op == 0 ? raw_a[2 * q + 1] : raw_b[2 * q + 1];
        u32x4_t w[3];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          // (copies: a bit cast of a vector's element itself reads the vector's first)
          const uint32_t u0 = e < 2 ? lo[2 * e] : hi[2 * e - 4], u1 = e < 2 ? lo[2 * e + 1] : hi[2 * e - 3];
          uint32_t parts[3];
          split3(__builtin_bit_cast(float, u0), __builtin_bit_cast(float, u1), parts);
#pragma unroll
          for (int s = 0; s < 3; ++s) w[s][e] = parts[s];
        }
#pragma unroll
        for (int s = 0; s < 3; ++s) *(u32x4_t*)(lds + (3 * op + s) * PART + w_off + q * 16 * tp::SIDE) = w[s];
      }
  };

  int a_rd[4], b_rd[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    a_rd[i] = tp::frag_offset(lane, wave_m * 4 + i);
    b_rd[i] = 3 * PART + tp::frag_offset(lane, wave_n * 4 + i);
  }
  auto frags = [&](const int (&rd)[4], int part, s16x8_t* f) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const unsigned short* p = lds + rd[i] + part * PART;
      f[i] = __builtin_shufflevector(lds_read_tr(p), lds_read_tr(p + 4 * tp::SIDE), 0, 1, 2, 3, 4, 5, 6, 7);
    }
  };
  f32x4_t acc[4][4], low[4][4];   // the products of the first parts; all others
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = low[i][j] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
  auto products = [&](f32x4_t (&c)[4][4], const s16x8_t* fa, const s16x8_t* fb) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        c[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, fb[j]), __builtin_bit_cast(bf16x8_t, fa[i]), c[i][j], 0, 0, 0);
  };

  const int nk = (T + 31) / 32;
  fetch();
  stage();
  fetch();
  __syncthreads();
  for (int k = 0; k < nk; ++k) {
    // (in an order that keeps at most five of the six operand parts in registers)
    s16x8_t a1[4], a2[4], a3[4], b1[4], b2[4], b3[4];
    frags(a_rd, 1, a2);
    frags(b_rd, 2, b3);
    frags(a_rd, 0, a1);
    products(low, a2, b3);
    frags(b_rd, 1, b2);
    products(low, a1, b3);
    frags(a_rd, 2, a3);
    products(low, a1, b2);
    products(low, a2, b2);
    frags(b_rd, 0, b1);
    products(low, a3, b2);
    products(low, a3, b1);
    products(low, a2, b1);
    products(acc, a1, b1);
    __syncthreads();    // every wave has read its fragments
    if (k + 1 < nk) {
      stage();
      fetch();
      __syncthreads();
    }
  }

#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = (acc[i][j] + low[i][j]) * F32x3Cfg::UNSCALE;

  // acc[i][j][r] = element (64 wave_m + 16 i + lane % 16, 64 wave_n + 16 j + 4 (lane / 16) + r) of the tile
  auto square_sum = [&]() {
    float ss[4] = {0.0f, 0.0f, 0.0f, 0.0f};   // short chains: a norm's rounding is its whole sample's
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) ss[j] = fmaf(acc[i][j][e], acc[i][j][e], ss[j]);
    return (ss[0] + ss[1]) + (ss[2] + ss[3]);
  };
  float ss = square_sum();
  if (__syncthreads_or(!(ss <= 3.0e38f))) {
    const int m = m0 + 64 * wave_m + (lane & 15), n = n0 + 64 * wave_n + 4 * (lane >> 4);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    // an operand that is not finite meets the zeros beyond a ragged edge of the tiles that the layer is planned on, 256 x 256 for the
    // fp32 matrix instructions and 64 x 64 for the generic kernel, which makes the norm NaN: likewise (EDGE_ bits)
    const bool edge_d = (a.edges & EDGE_LARGE_D) && tm == a.tiles_m - 1, edge_p = (a.edges & EDGE_LARGE_P) && tn == a.tiles_n - 1;
    float ragged = 0.0f;
#pragma unroll 1
    for (int t = 0; t < T; ++t) {
      float y[4];
      f32x4_t x[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) y[i] = m + 16 * i < D ? ((const float*)pa)[(size_t)t * D + m + 16 * i] : 0.0f;
#pragma unroll
      for (int j = 0; j < 4; ++j) x[j] = n + 16 * j < P ? *(const f32x4_t*)((const float*)pb + (size_t)t * P + n + 16 * j) : f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        ragged = fmaf(0.0f, edge_p ? y[i] : 0.0f, ragged);
#pragma unroll
        for (int e = 0; e < 4; ++e) ragged = fmaf(0.0f, edge_d ? x[i][e] : 0.0f, ragged);
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[i][j][e] = fmaf(y[i], x[j][e], acc[i][j][e]);
      }
    }
    ss = wave_outside(a.edges, m0 + 64 * wave_m, n0 + 64 * wave_n, D, P) ? 0.0f : square_sum() + ragged;
  }
  float* const red = (float*)lds + 64 * F32x3Cfg::OUT_PITCH;
  const float w = wave_sum_to_lane63(ss);
  if (lane == 63) red[wave] = w;
  float* const st = (float*)lds;
  float* const out = (float*)a.scratch + (size_t)sample * D * P;
#pragma unroll 1
  for (int h = 0; h < 2; ++h) {   // 64 rows at a time through LDS, so that whole rows are written
    if (wave_m == h) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          *(f32x4_t*)(st + (16 * i + (lane & 15)) * F32x3Cfg::OUT_PITCH + 64 * wave_n + 16 * j + 4 * (lane >> 4)) = acc[i][j];
    }
    __syncthreads();
    if (h == 0 && tid == 0) a.partials[(size_t)sample * tiles + tile] = (red[0] + red[1]) + (red[2] + red[3]);
#pragma unroll
    for (int it = 0; it < 8; ++it) {
      const int r = (tid >> 5) + 8 * it, row = m0 + 64 * h + r, col = n0 + 4 * (tid & 31);
      if (row < D && col < P) *(f32x4_t*)(out + (size_t)row * P + col) = *(const f32x4_t*)(st + r * F32x3Cfg::OUT_PITCH + 4 * (tid & 31));
    }
    __syncthreads();
  }
}

}  // namespace flashdp
