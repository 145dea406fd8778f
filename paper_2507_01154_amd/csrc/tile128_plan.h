// Index arithmetic of the 128 x 128 direct-to-LDS kernels (gemm_tile128.hip.h), kept apart from them so that a host
// compiler can check it.  The hardware facts are those of lds_plan.h (a wave-wide 16-byte-per-lane direct load writes 1 KB
// of LDS, lane L's bytes at destination + 16 L; the lane pattern of ds_read_b64_tr_b16), the fragments and the swizzle those
// of lds_plan16.h (v_mfma_f32_16x16x32), for operand tiles of 32 (t) rows of 128 elements (256 bytes, one turn of the LDS
// banks): the 16-byte chunk c of row t is kept at position c ^ (((t & 3) << 2) | (((t >> 3) & 1) << 1)), which sends the
// eight 32-byte windows that 32 lanes of a transposed read touch (rows t..t+3 and t+8..t+11 of one 16-wide block) to eight
// different bank groups.
#pragma once
#include <stdint.h>

#include "lds_plan.h"

namespace flashdp {
namespace tile128_plan {

constexpr int SIDE = 128;           // elements per tile row of either operand
constexpr int TILE_ROWS = 32;       // k-tile depth
constexpr int WAVES = 4;
constexpr int STAGES = 4;
constexpr int OPERAND_ELEMS = TILE_ROWS * SIDE;

// element offset of operand `operand` (0 = dY, 1 = X) of ring stage `stage`: operand-major, so that a fragment read
// reaches every stage through the 16-bit offset field
FLASHDP_PLAN_HD int tile_base(int stage, int operand) { return (operand * STAGES + stage) * OPERAND_ELEMS; }

FLASHDP_PLAN_HD int swizzle(int t) { return ((t & 3) << 2) | (((t >> 3) & 1) << 1); }

// Direct loads: instruction q (0 or 1) of wave w fills tile rows 16 q + 4 w .. + 3 of an operand.
FLASHDP_PLAN_HD int load_row(int wave, int lane) { return 4 * wave + (lane >> 4); }   // add 16 q
// the chunk of that row the lane fetches (rows + 16 have the same swizzle)
FLASHDP_PLAN_HD int load_chunk(int wave, int lane) { return (lane & 15) ^ swizzle(load_row(wave, lane)); }
FLASHDP_PLAN_HD uint32_t load_dst_bytes(int stage, int operand, int wave, int q) {
  return (uint32_t)(tile_base(stage, operand) + (16 * q + 4 * wave) * SIDE) * 2u;
}

// Where element (row, col) of an operand tile is kept, in elements from the start of that tile.
FLASHDP_PLAN_HD int kept_at(int row, int col) { return row * SIDE + (((col >> 3) ^ swizzle(row)) << 3) + (col & 7); }

// Transposed fragment reads of one k-tile: 4 contiguous elements at tile row frag_row (and + 4 for the second read, which
// keeps the swizzle), columns 16 block + frag_col .. + 3.
FLASHDP_PLAN_HD int frag_row(int lane) { return 8 * (lane >> 4) + ((lane & 15) >> 2); }
FLASHDP_PLAN_HD int frag_col(int lane) { return 4 * (lane & 3); }
FLASHDP_PLAN_HD int frag_offset(int lane, int block) { return kept_at(frag_row(lane), 16 * block + frag_col(lane)); }

}  // namespace tile128_plan
}  // namespace flashdp
