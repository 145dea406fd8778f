// Contraction on 128 x 128 tiles that walks over several samples without draining its pipeline: the two passes of the
// two-pass schedule for short sequences, and, one sample a workgroup, the parking pass of layers whose 256 x 256 tiles are
// too few to fill the chip or end in a nearly empty round (the rule is in park_plan; 768 x 3072, B = 1, T = 1024, bf16: 14.8 us
// with tiles staged through registers, 11.5 so; B = 4: 31.6 on 256 x 256 tiles, 26.9).
//
// Why two passes.  With few tokens a per-sample gradient tile is a handful of k-tiles of work, and parking it (2 + 2 bytes an element
// and sample, beside 4 T / 1e15 seconds of arithmetic) is most of the time, the rest being start and end of one workgroup per
// tile and sample.  Computing every G_i twice costs 2 T FLOP an element and sample instead and nothing is parked; and a
// workgroup that keeps its tile and walks over the samples loads the next sample's first k-tiles while it multiplies the
// last ones of this sample (the accumulating pass up to 64 tokens; see in_step).  Every term stays in fp32, where parking rounds it to 8 bits once.
//
// Pipeline as gemm_mfma_dma_kernel: operand tiles straight into a ring of 4 LDS stages, the loads of k-tile k + 3 issued
// at the top of k-tile k, one barrier per k-tile, waits for the direct loads by hand (they complete in order).  4 waves of
// 64 x 64 on v_mfma_f32_16x16x32, 64 KB of LDS: two workgroups per CU, so that one's barriers and sample boundaries are
// covered by the other's matrix-core work.
//
// Bound by the issue path of one wave between two barriers, not by a rate (matrix cores busy 0.45, LDS 0.25, a fifth ring
// stage gains nothing): hence fragment reads and direct loads in the shadow of the matrix instructions, LDS stages as
// compile-time constants, cursors moved on by additions.  Norm pass of 4096 x 4096, bf16, B = 2, T = 2048: 1.19 PFLOP/s (1.07
// with the reads in front of the products), B = 16, T = 128: 0.96; accumulating pass with its noise 0.98 and 0.69.
// A GPT-2 block, B = 32, T = 128, fp16: 279 us a call parked, 148 so.  A CU takes direct loads at about 30 bytes a clock, which is
// what a workgroup by itself runs at (768 x 3072, B = 1).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "elementwise.hip.h"
#include "gemm_mfma.hip.h"
#include "gemm_mfma_dma.hip.h"
#include "gemm_mfma_dma16.hip.h"
#include "tile128_plan.h"

namespace flashdp {

// What the tiles that a layer is planned on have at its edges and 128 x 128 tiles have not, or the other way round: an operand that
// is not finite and meets the zeros beyond an edge makes the norm NaN, which poisons the output, where it would be infinite
// otherwise and the factor 0.  Which tiles a layer takes must not decide that.
enum { EDGE_LARGE_D = 1, EDGE_LARGE_P = 2,   // larger tiles reach beyond D, beyond P (any_not_finite)
       EDGE_ONLY_D = 4, EDGE_ONLY_P = 8 };   // 128 x 128 tiles reach beyond D, P and the plan's do not (odd multiples of 64; wave_outside)

struct Tile128Layer {
  const void* X;         // [B][T][P]
  const void* dY;        // [B][T][D]
  int B, T, P, D;
  int tiles_m, tiles_n;  // ceil(D / 128), ceil(P / 128)
  int edges;             // EDGE_ bits
  int splits;            // workgroups per tile: split r walks over samples [B r / splits, B (r + 1) / splits)
  float* partials;       // squared-norm partial sums: [B][tiles_m * tiles_n][4], one per wave (NORM); [B][tiles_m * tiles_n] (SPILL)
  void* scratch;         // [B][D][P] bfloat16 (SPILL)
  const float* factors;  // [B] clip factors (ACCUM)
  float* out;            // [D][P], or fp32 partial sums [splits][D][P] where splits > 1 (ACCUM)
  float noise_scale;     // added by the kernel itself where splits == 1
  int accumulate;
  uint64_t seed;
  uint32_t layer;
};
struct Tile128Args {
  int n;
  int first[GROUP_MAX + 1];   // workgroups first[l] .. first[l + 1] - 1 are layer l's; multiples of 8 (see xcd_remap)
  Tile128Layer layer[GROUP_MAX];
};

// The layer that this workgroup belongs to, and which of the layer's workgroups it is.  A layer by itself is passed by
// itself (parking pass): eight layers' arguments are a kilobyte, which the host takes 0.6 us longer to hand over, and small calls in
// a row are bound by the host (16 x 648, f16, B = 1, T = 8: 11.8 us a call, 11.2 so; 768 x 768, bf16, B = 1, T = 1024: 15.2, 14.6).
__device__ __forceinline__ const Tile128Layer& layer_of(const Tile128Layer& a, int* bid) {
  *bid = blockIdx.x;
  return a;
}
__device__ __forceinline__ const Tile128Layer& layer_of(const Tile128Args& g, int* bid) {
  const int l = group_of(g.first, g.n, blockIdx.x);
  *bid = (int)blockIdx.x - g.first[l];
  return g.layer[l];
}

struct Tile128Cfg {
  static constexpr int NT = 256;
  static constexpr int LDS_BYTES = 2 * tile128_plan::STAGES * tile128_plan::OPERAND_ELEMS * 2;   // 64 KB
  static constexpr int OUT_PITCH = 128 + 4;                                                      // floats; 64 rows at a time are staged
  static constexpr int PARK_PITCH = 128 + 8;                                                     // 16-bit elements: 16-byte aligned rows
  static_assert(64 * OUT_PITCH * 4 <= LDS_BYTES && 128 * PARK_PITCH * 2 + 16 <= LDS_BYTES, "output rows fit the ring");
};

// The first product of a sample: c = a b.  As mfma16_inplace the accumulators are outputs of inline assembly, so that they
// stay where they are (with the builtin two sets of them alternate, and the totals no longer fit the registers); the
// waits between the matrix cores and a vector-ALU access are by hand.
template <int DT>
__device__ __forceinline__ void mfma16_first(f32x4_t& c, const s16x8_t& a, const s16x8_t& b) {
  if constexpr (DT == DT_BF16) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=&v"(c) : "v"(a), "v"(b));
  } else {
    asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, 0" : "=&v"(c) : "v"(a), "v"(b));
  }
}

// Sum over the 64 lanes, the same bits in every lane's chain of additions each time (lane 63 holds the result).
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float add_dpp(float v) {
  const int m = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, ROW_MASK, 0xF, false);
  return v + __builtin_bit_cast(float, m);
}
__device__ __forceinline__ float wave_sum_to_lane63(float v) {
  v = add_dpp<0x111, 0xF>(v);   // row_shr:1
  v = add_dpp<0x112, 0xF>(v);   // row_shr:2
  v = add_dpp<0x114, 0xF>(v);   // row_shr:4
  v = add_dpp<0x118, 0xF>(v);   // row_shr:8: lane 15 of each row of 16 holds the row's sum
  v = add_dpp<0x142, 0xA>(v);   // row_bcast:15 into rows 1 and 3
  v = add_dpp<0x143, 0xC>(v);   // row_bcast:31 into rows 2 and 3
  return v;
}

// EDGE_ONLY_D, EDGE_ONLY_P: whether all of a wave's 64 x 64 elements from (m, n) on lie beyond such an edge, where its squares do not
// count.  (They are zero unless an operand is not finite.)
__device__ __forceinline__ bool wave_outside(int edges, int m, int n, int D, int P) {
  return ((edges & EDGE_ONLY_D) && m >= D) || ((edges & EDGE_ONLY_P) && n >= P);
}

// EDGE_LARGE_D, EDGE_LARGE_P: a norm that is infinite has its operands looked through: whether any of
// rows x 8 chunks elements, a row every `pitch` elements, is not finite (the share of thread `me` of N, in rows of N_CHUNKS chunks).
template <int DT, int N, int N_CHUNKS>
__device__ __forceinline__ bool any_not_finite(const unsigned short* p, int64_t rows, int chunks, int64_t pitch, int me) {
  constexpr uint32_t EXP = DT == DT_BF16 ? 0x7F807F80u : 0x7C007C00u;
  bool found = false;
  for (int c = me % N_CHUNKS; c < chunks; c += N_CHUNKS)
#pragma unroll 4
    for (int64_t r = me / N_CHUNKS; r < rows; r += N / N_CHUNKS) {
      const u32x4_t v = *(const u32x4_t*)(p + r * pitch + 8 * c);
#pragma unroll
      for (int q = 0; q < 4; ++q)
        found |= (v[q] & EXP & 0xFFFFu) == (EXP & 0xFFFFu) || (v[q] & EXP & 0xFFFF0000u) == (EXP & 0xFFFF0000u);
    }
  return found;
}

template <int MODE, int DT, typename Args = Tile128Args>
__global__ __launch_bounds__(256, 2) void gemm_tile128_kernel(const Args g) {
  static_assert(MODE == MODE_NORM || MODE == MODE_ACCUM || MODE == MODE_SPILL, "the passes this tiling has");
  namespace tp = tile128_plan;
  constexpr int STAGES = tp::STAGES;
  extern __shared__ __attribute__((aligned(16))) unsigned short lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wave_m = wave & 1, wave_n = wave >> 1;

  int bid;
  const Tile128Layer& a = layer_of(g, &bid);
  const int tiles = a.tiles_m * a.tiles_n, total = tiles * a.splits;
  if (bid >= total) return;   // the whole workgroup, before any barrier
  const int item = xcd_remap(bid, total);
  const int split = item / tiles, tile = item - split * tiles;
  const int s_begin = (int)((int64_t)a.B * split / a.splits), s_end = (int)((int64_t)a.B * (split + 1) / a.splits);
  int tm, tn;
  tile_coords<8>(tile, a.tiles_m, a.tiles_n, &tm, &tn);
  const int m0 = tm * tp::SIDE, n0 = tn * tp::SIDE;

  // ---- direct-load plan (out-of-range columns are sent to 2 GiB, beyond num_records, and read as zeros)
  const int d_row = tp::load_row(wave, lane), d_chunk = tp::load_chunk(wave, lane);
  const bool a_ok = m0 + d_chunk * 8 < a.D, b_ok = n0 + d_chunk * 8 < a.P;
  const uint32_t a_off0 = a_ok ? (uint32_t)(d_row * a.D + m0 + d_chunk * 8) * 2u : 0x80000000u;
  const uint32_t b_off0 = b_ok ? (uint32_t)(d_row * a.P + n0 + d_chunk * 8) * 2u : 0x80000000u;
  const uint32_t a_half = (uint32_t)(16 * a.D) * 2u, b_half = (uint32_t)(16 * a.P) * 2u;
  const uint32_t a_kstep = 2u * a_half, b_kstep = 2u * b_half;
  const uint32_t a_bytes = (uint32_t)a.T * (uint32_t)a.D * 2u, b_bytes = (uint32_t)a.T * (uint32_t)a.P * 2u;
  const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned short*)lds;
  const int kt_per_sample = (a.T + 31) / 32;

  // Fetch cursor: descriptors of the sample and byte offsets of the k-tile to load next, moved on from k-tile to k-tile.
  // Past the last tile it stays with the last sample, at rows >= T, which read as zeros.
  u32x4_t rsa = make_rsrc_words((const char*)a.dY + (size_t)s_begin * a_bytes, a_bytes);
  u32x4_t rsb = make_rsrc_words((const char*)a.X + (size_t)s_begin * b_bytes, b_bytes);
  uint32_t a_off = a_off0, b_off = b_off0;
  int ld_left = kt_per_sample, ld_samples = s_end - s_begin;
  auto advance = [&]() {
    a_off += a_kstep;
    b_off += b_kstep;
    if (--ld_left == 0 && --ld_samples > 0) {
      const uint64_t na = (((uint64_t)rsa[1] << 32) | rsa[0]) + a_bytes, nb = (((uint64_t)rsb[1] << 32) | rsb[0]) + b_bytes;
      rsa[0] = (uint32_t)na; rsa[1] = (uint32_t)(na >> 32);
      rsb[0] = (uint32_t)nb; rsb[1] = (uint32_t)(nb >> 32);
      a_off = a_off0;
      b_off = b_off0;
      ld_left = kt_per_sample;
    }
  };
  auto load_part = [&](int stage, auto q_c) {
    constexpr int q = decltype(q_c)::value;
    if constexpr (q < 2) load_to_lds(rsa, a_off + q * a_half, lds_base + tp::load_dst_bytes(stage, 0, wave, q));
    else load_to_lds(rsb, b_off + (q - 2) * b_half, lds_base + tp::load_dst_bytes(stage, 1, wave, q - 2));
  };

  int a_rd[4], b_rd[4];   // element offsets of the wave's fragments in stage 0
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    a_rd[i] = tp::tile_base(0, 0) + tp::frag_offset(lane, wave_m * 4 + i);
    b_rd[i] = tp::tile_base(0, 1) + tp::frag_offset(lane, wave_n * 4 + i);
  }
  s16x8_t fa[2][4], fb[2][4];
  // read r (0..15) of a k-tile's fragments: half r % 2 of X block r / 2, then of dY block r / 2 - 4
  s16x4_t half_frag;
  auto read_frag = [&](int stage, auto r_c, s16x8_t* pfa, s16x8_t* pfb) {
    constexpr int r = decltype(r_c)::value, f = (r / 2) % 4;
    const unsigned short* p = lds + stage * tp::OPERAND_ELEMS + (r < 8 ? b_rd[f] : a_rd[f]) + (r % 2) * 4 * tp::SIDE;
    const s16x4_t v = lds_read_tr(p);
    if constexpr (r % 2 == 0) half_frag = v;
    else (r < 8 ? pfb : pfa)[f] = __builtin_shufflevector(half_frag, v, 0, 1, 2, 3, 4, 5, 6, 7);
  };

  f32x4_t acc[4][4];
  f32x4_t tot[MODE == MODE_ACCUM ? 4 : 1][MODE == MODE_ACCUM ? 4 : 1];
  const f32x4_t zero4 = {0.0f, 0.0f, 0.0f, 0.0f};
  if constexpr (MODE == MODE_ACCUM) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) tot[i][j] = zero4;
  }

  const bool outside = wave_outside(a.edges, m0 + 64 * wave_m, n0 + 64 * wave_n, a.D, a.P);

  // End of a sample: its squared norm is noted (NORM), or its clipped gradient joins the total (ACCUM).  Totals of their own,
  // so that no sample's products are added to a large sum one by one and a clip factor of 0 is harmless.  Lane q holds the
  // sum of this wave's squares resp. the clip factor of sample s_base + q, so that memory is met once in 64 samples: a store
  // per sample stood in the queue of the direct loads, whose waits are in order, until it was acknowledged.
  int s = s_begin, s_base = s_begin, left = kt_per_sample;   // the sample in progress and its k-tiles to come
  float per_lane = 0.0f;
  auto lanes_to_memory = [&]() {   // NORM: samples s_base .. s - 1
    if (s_base + lane < s) a.partials[((size_t)(s_base + lane) * tiles + tile) * 4 + wave] = per_lane;
  };
  auto lanes_from_memory = [&]() { per_lane = a.factors[min(s_base + lane, a.B - 1)]; };
  // The compiler waits here for the load above, and not where the value is used: as it does not see the direct loads, that would
  // be a wait for all of them at every sample.  Such a wait is worth its time where a sample has more than two k-tiles: without it the
  // workgroups that share operands drift apart, and the loads they run ahead with come from farther away.  bf16, a call, with a
  // wait at every sample and without: 4096 x 4096, T = 16, B = 64: 189 us, 179; a GPT-2 block, B = 256, T = 16: 337, 315, T = 64: 597, 593,
  // T = 128: 1176, 1271; 4096 x 4096, B = 128, T = 192: 1831, 2073; 1024 x 4096, B = 200, T = 128: 420, 414.
  const bool in_step = a.T > 64;
  auto lanes_arrived = [&]() { asm volatile("" : "+v"(per_lane)); };
  if constexpr (MODE == MODE_ACCUM) lanes_from_memory();
  auto sample_done = [&]() {
    if constexpr (MODE == MODE_NORM) {
      float ss[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) ss[e] = fmaf(acc[i][j][e], acc[i][j][e], ss[e]);
      const float w = wave_sum_to_lane63((ss[0] + ss[1]) + (ss[2] + ss[3]));
      const float sum = outside ? 0.0f : __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, w), 63));
      per_lane = lane == s - s_base ? sum : per_lane;
    } else if constexpr (MODE == MODE_ACCUM) {
      if (in_step) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      const float c = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, per_lane), s - s_base));
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) tot[i][j][e] = fmaf(c, acc[i][j][e], tot[i][j][e]);
    }
    ++s;
    left = kt_per_sample;
    if (s - s_base == 64) {
      if constexpr (MODE == MODE_NORM) lanes_to_memory();
      s_base = s;
      if constexpr (MODE == MODE_ACCUM) { lanes_from_memory(); lanes_arrived(); }
    }
  };

  // One k-tile, whose fragments are in registers, from stage `cur`; false after the last one.  At its top the next k-tile is
  // in LDS (every wave's loads of it have landed) and every wave has read stage `cur`, which the loads of k-tile k + 4 may
  // refill.  The reads of the next k-tile's fragments and those loads are spread over this one's matrix instructions, in
  // whose shadow (16 cycles each) they issue; in front of them they kept the matrix cores waiting.
  auto k_tile = [&](auto cur_c) -> bool {
    constexpr int cur = decltype(cur_c)::value, p = cur & 1;
    asm volatile("s_waitcnt vmcnt(8) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    auto products = [&](auto first_c) {
      static_for<16>([&](auto m_c) {
        constexpr int m = decltype(m_c)::value, i = m / 4, j = m % 4;
        if constexpr (decltype(first_c)::value) mfma16_first<DT>(acc[i][j], fb[p][j], fa[p][i]);
        else mfma16_inplace<DT>(acc[i][j], fb[p][j], fa[p][i]);
        if constexpr (m < 8) {
          read_frag((cur + 1) % STAGES, std::integral_constant<int, 2 * m>{}, fa[p ^ 1], fb[p ^ 1]);
          read_frag((cur + 1) % STAGES, std::integral_constant<int, 2 * m + 1>{}, fa[p ^ 1], fb[p ^ 1]);
        } else if constexpr (m < 12) {
          load_part(cur, std::integral_constant<int, m - 8>{});
        }
        __builtin_amdgcn_sched_barrier(0);
      });
    };
    if (left == kt_per_sample) products(std::true_type{});   // a sample's first products start from zero
    else products(std::false_type{});
    advance();
    if (--left == 0) {
      matrix_core_results_settle();
      sample_done();
      return s < s_end;
    }
    return true;
  };

#pragma unroll
  for (int st = 0; st < STAGES; ++st) {
    static_for<4>([&](auto q_c) { load_part(st, q_c); });
    advance();
  }
  asm volatile("s_waitcnt vmcnt(12)\n\ts_barrier" ::: "memory");
  if constexpr (MODE == MODE_ACCUM) lanes_arrived();
  static_for<16>([&](auto r_c) { read_frag(0, r_c, fa[0], fb[0]); });
  for (;;) {
    if (!k_tile(std::integral_constant<int, 0>{})) break;
    if (!k_tile(std::integral_constant<int, 1>{})) break;
    if (!k_tile(std::integral_constant<int, 2>{})) break;
    if (!k_tile(std::integral_constant<int, 3>{})) break;
  }
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");   // loads past the end still write zeros into LDS

  if constexpr (MODE == MODE_NORM) lanes_to_memory();
  if constexpr (MODE == MODE_SPILL) {
    // One sample (splits == B).  The tile leaves in bfloat16 through LDS, in whole rows, and its squared norm is taken as parked
    // (see tile_epilogue).  acc[i][j][r] = element (64 wave_m + 16 i + lane % 16, 64 wave_n + 16 j + 4 (lane / 16) + r) of the tile.
    constexpr int EP = Tile128Cfg::PARK_PITCH;
    float* const red = (float*)(lds + 128 * EP);
    unsigned short* const st = lds + (64 * wave_m + (lane & 15)) * EP + 64 * wave_n + 4 * (lane >> 4);
    float ss = 0.0f;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        uint2 v;
        v.x = pack2_16bit<DT_BF16>(acc[i][j][0], acc[i][j][1]);
        v.y = pack2_16bit<DT_BF16>(acc[i][j][2], acc[i][j][3]);
        const float r0 = __builtin_bit_cast(float, v.x << 16), r1 = __builtin_bit_cast(float, v.x & 0xFFFF0000u);
        const float r2 = __builtin_bit_cast(float, v.y << 16), r3 = __builtin_bit_cast(float, v.y & 0xFFFF0000u);
        ss = fmaf(r0, r0, ss); ss = fmaf(r1, r1, ss); ss = fmaf(r2, r2, ss); ss = fmaf(r3, r3, ss);
        *(uint2*)(st + (i * 16) * EP + j * 16) = v;
      }
    float w = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, wave_sum_to_lane63(ss)), 63));
    if (outside) w = 0.0f;
    if (__builtin_expect(w == __builtin_inff(), 0)) {   // of this wave's 64 x 64 elements
      const int m = m0 + 64 * wave_m, n = n0 + 64 * wave_n;
      bool found = false;
      if (a.edges & EDGE_LARGE_D) found |= any_not_finite<DT, 64, 8>((const unsigned short*)a.X + (size_t)s_begin * a.T * a.P + n, a.T, min(8, (a.P - n) / 8), a.P, lane);
      if (a.edges & EDGE_LARGE_P) found |= any_not_finite<DT, 64, 8>((const unsigned short*)a.dY + (size_t)s_begin * a.T * a.D + m, a.T, min(8, (a.D - m) / 8), a.D, lane);
      if (__any(found)) w = __builtin_nanf("");
    }
    if (lane == 63) red[wave] = w;
    __syncthreads();
    if (tid == 0) a.partials[(size_t)s_begin * tiles + tile] = (red[0] + red[1]) + (red[2] + red[3]);
    unsigned short* const sc = (unsigned short*)a.scratch + (size_t)s_begin * a.D * a.P;
#pragma unroll
    for (int it = 0; it < 8; ++it) {
      const int r = (tid >> 4) + 16 * it, row = m0 + r, col = n0 + 8 * (tid & 15);
      if (row < a.D && col < a.P)   // P is a multiple of 8 on this path: a chunk is all in or all out
        __builtin_nontemporal_store(*(const u32x4_t*)(lds + r * EP + 8 * (tid & 15)), (u32x4_t*)(sc + (size_t)row * a.P + col));
    }
  }
  if constexpr (MODE == MODE_ACCUM) {
    // tot[i][j][r] = element (m0 + 64 wave_m + 16 i + lane % 16, n0 + 64 wave_n + 16 j + 4 (lane / 16) + r).  64 rows at a
    // time go through LDS, so that whole rows are written and the noise generator stands in one loop.
    float* const stage = (float*)lds;
    constexpr int OP = Tile128Cfg::OUT_PITCH;
    float* const out = a.splits > 1 ? a.out + (size_t)split * a.D * a.P : a.out;
    const float noise_scale = a.splits > 1 ? 0.0f : a.noise_scale;
    const bool add = a.splits == 1 && a.accumulate != 0;
#pragma unroll 1
    for (int h = 0; h < 2; ++h) {
      if (wave_m == h) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j)
            *(f32x4_t*)(stage + (16 * i + (lane & 15)) * OP + 64 * wave_n + 16 * j + 4 * (lane >> 4)) = tot[i][j];
      }
      __syncthreads();
#pragma unroll 1
      for (int c = tid; c < 64 * 32; c += 256) {
        const int r = c >> 5, row = m0 + 64 * h + r, col = n0 + 4 * (c & 31);
        if (row >= a.D || col >= a.P) continue;   // P is a multiple of 8 on this path: a group of 4 is all in or all out
        f32x4_t v = *(const f32x4_t*)(stage + r * OP + 4 * (c & 31));
        const size_t e = (size_t)row * a.P + col;
        if (noise_scale != 0.0f) {
          const Normals4 z = noise_group(a.seed, a.layer, e >> 2);
#pragma unroll
          for (int q = 0; q < 4; ++q) v[q] = fmaf(noise_scale, z.z[q], v[q]);
        }
        if (add) {
          const f32x4_t o = *(const f32x4_t*)(out + e);
          v += o;
        }
        __builtin_nontemporal_store(v, (f32x4_t*)(out + e));
      }
      __syncthreads();
    }
  }
}

// n_i and c_i from the partials of gemm_tile128_kernel, one workgroup per sample and layer; fixed order of additions.
struct Tile128ClipArgs {
  int n, B, T;
  struct Layer { const float* partials; float* factors; float* out_norms; int per_sample; float C; const void* X; const void* dY; int P, D, edges; } layer[GROUP_MAX];
};
template <int DT>
__global__ __launch_bounds__(256) void tile128_clip_kernel(const Tile128ClipArgs g) {
  __shared__ double red[4];
  const int l = blockIdx.x / g.B, i = blockIdx.x - l * g.B, tid = threadIdx.x;
  const Tile128ClipArgs::Layer& a = g.layer[l];
  const float4* p = (const float4*)(a.partials + (size_t)i * a.per_sample);   // four waves' sums per tile
  double s = 0.0;
#pragma unroll 4
  for (int k = tid; k < a.per_sample / 4; k += 256) {
    const float4 v = p[k];
    s += ((double)v.x + (double)v.y) + ((double)v.z + (double)v.w);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
  if ((tid & 63) == 0) red[tid >> 6] = s;
  __syncthreads();
  double n = sqrt((red[0] + red[1]) + (red[2] + red[3]));
  if ((a.edges & (EDGE_LARGE_D | EDGE_LARGE_P)) && n == __builtin_inf()) {
    bool found = false;
    if (a.edges & EDGE_LARGE_D) found |= any_not_finite<DT, 256, 16>((const unsigned short*)a.X + (size_t)i * g.T * a.P, g.T, a.P / 8, a.P, tid);
    if (a.edges & EDGE_LARGE_P) found |= any_not_finite<DT, 256, 16>((const unsigned short*)a.dY + (size_t)i * g.T * a.D, g.T, a.D / 8, a.D, tid);
    if (__syncthreads_or(found)) n = __builtin_nan("");
  }
  if (tid == 0) {
    a.factors[i] = clip_factor_of(n, a.C);
    if (a.out_norms) a.out_norms[i] = (float)n;
  }
}

// out = (accumulate ? out : 0) + sum over splits of the partial sums + noise.
struct Tile128SumArgs {
  int n;
  int first[GROUP_MAX + 1];
  struct Layer { const float* partial; float* out; size_t S; int splits, accumulate; float noise_scale; uint64_t seed; uint32_t layer; } layer[GROUP_MAX];
};
__global__ __launch_bounds__(256) void tile128_sum_kernel(const Tile128SumArgs g) {
  const int l = group_of(g.first, g.n, blockIdx.x);
  const Tile128SumArgs::Layer& a = g.layer[l];
  const size_t v = (size_t)((int)blockIdx.x - g.first[l]) * 256 + threadIdx.x;
  if (4 * v >= a.S) return;   // S is a multiple of 8
  f32x4_t acc = a.accumulate ? ((const f32x4_t*)a.out)[v] : f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 4
  for (int q = 0; q < a.splits; ++q) acc += ((const f32x4_t*)(a.partial + (size_t)q * a.S))[v];
  if (a.noise_scale != 0.0f) {
    const Normals4 z = noise_group(a.seed, a.layer, v);
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[q] = fmaf(a.noise_scale, z.z[q], acc[q]);
  }
  __builtin_nontemporal_store(acc, (f32x4_t*)a.out + v);
}

}  // namespace flashdp
