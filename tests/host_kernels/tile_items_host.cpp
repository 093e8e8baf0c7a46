// The items of a tile (tile_item of step_common.hpp) and the boundary map of a
// stencil node (bc_node32 of physics.hpp) on the CPU, at sizes up to the largest
// that the library takes, where a tile's end and a node's number do not fit an int.
// Prints the wrong ones and the number looked at.
#include "hip/hip_runtime.h"

thread_local dim3s threadIdx, blockIdx;
dim3s gridDim, blockDim;
pthread_barrier_t g_block_barrier;
#define __builtin_amdgcn_readfirstlane(v) (v)
#include "step_common.hpp"

using namespace acat;

int main() {
  const int64_t top = ((int64_t)1 << 31) - 2;   // most interfaces of a 1D problem
  long bad = 0, seen = 0;
  for (int T : {1, 7, 39, 127, 240, 255, 256})
    for (int64_t n : {(int64_t)1, (int64_t)255, (int64_t)1000, top - 300, top - 126, top - 125, top - 1, top}) {
      const int64_t tiles = (n + T - 1) / T;
      for (int64_t tile : {(int64_t)0, tiles / 2, tiles - 1})
        for (int lane = 0; lane < 256; ++lane, ++seen) {
          const __int128 k = (__int128)tile * T + lane;
          bad += tile_item((uint32_t)tile, T, lane, n) != (lane < T && k < n ? (int64_t)k : -1);
        }
    }
  for (int bc : {PERIODIC, TRANSMISSIVE})
    for (int64_t n : {(int64_t)12, (int64_t)13, top - 1})
      for (int64_t i = -1; i < n; i = i == 20 && n > 100 ? n - 20 : i + 1)
        for (int off = -6; off <= 6; ++off, ++seen)
          if (bc == TRANSMISSIVE || i >= 0) bad += bc_node32((int)i, off, (int)n, bc) != bc_index(i + off, n, bc);
  std::printf("%ld %ld\n", bad, seen);
  return 0;
}
