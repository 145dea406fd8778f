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

constexpr int WALK_STEP = 1024;   // elements of a row that one step of a workgroup of 256 threads takes

// f(k) for every step of one thread through a row of n elements; the thread's elements of the step are
// k, k + 256, k + 512, k + 768 as far as they are below n.
template <typename F>
FLASHDP_EP_HD void walk_row(int n, int thread, F f) {
  for (uint32_t k = (uint32_t)thread; k < (uint32_t)n; k += WALK_STEP) f(k);
}

}  // namespace edge_plan
}  // namespace flashdp
