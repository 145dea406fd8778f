// Index arithmetic at the ends of very long rows, kept apart from the kernels so that a host compiler can check it:
// features go up to 2^31 - 1, so an index one step past the last row element does not fit an int.
#pragma once
#include <stdint.h>

#if defined(__HIPCC__)
#define FLASHDP_EP_HD __host__ __device__ __forceinline__
#else
#define FLASHDP_EP_HD static inline
#endif

namespace flashdp {
namespace edge_plan {

// Tiles of the given side that cover n elements.
FLASHDP_EP_HD int tiles(int n, int side) { return (int)(((int64_t)n + side - 1) / side); }

// Whether `width` elements from column col on, col < n, lie inside a row of n.
FLASHDP_EP_HD bool chunk_fits(int col, int n, int width) { return n - col >= width; }

constexpr int WALK_CHUNKS = 4;    // chunks of V elements that a thread takes in one step

// f(k) for every step of one of 256 threads through a row of n elements; the thread's elements of the step are
// k + 256 * V * q + 0..V-1 for q below WALK_CHUNKS, as far as they are below n.
template <int V, typename F>
FLASHDP_EP_HD void walk_row(int n, int thread, F f) {
  for (uint32_t k = (uint32_t)(thread * V); k < (uint32_t)n; k += 256 * V * WALK_CHUNKS) f(k);
}

}  // namespace edge_plan
}  // namespace flashdp
