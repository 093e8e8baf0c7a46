// The tiles of a batch (batch_tiles, batch_split) on the CPU: reads nprob and then n
// and P of every problem and the tile lengths of P = 1..4; prints the tiles and the
// slots.  With an argument: reads nprob, n, P and nvar of batches of equal problems and
// prints whether each goes by tiles.
#include "hip/hip_runtime.h"

#include <vector>

thread_local dim3s threadIdx, blockIdx;
dim3s gridDim, blockDim;
pthread_barrier_t g_block_barrier;
#include "batch_tiles.hpp"

int main(int argc, char**) {
  if (argc > 1) {
    int np, p, nvar;
    long v;
    while (std::scanf("%d %ld %d %d", &np, &v, &p, &nvar) == 4) {
      const std::vector<int64_t> n(np, v);
      const std::vector<int32_t> P(np, p);
      std::printf("%d\n", (int)acat::batch_split(np, n.data(), P.data(), nvar).by_tiles);
    }
    return 0;
  }
  int np = 0, T[acat::BATCH_PMAX + 1] = {};
  if (std::scanf("%d", &np) != 1) return 1;
  std::vector<int64_t> n(np);
  std::vector<int32_t> P(np), first(np, -1), count(np, -1);
  for (int b = 0; b < np; ++b) {
    long v = 0;
    if (std::scanf("%ld %d", &v, &P[b]) != 2) return 1;
    n[b] = v;
  }
  for (int p = 1; p <= acat::BATCH_PMAX; ++p)
    if (std::scanf("%d", &T[p]) != 1) return 1;
  int64_t nt = 0;
  for (int b = 0; b < np; ++b) nt += (n[b] + T[P[b]] - 1) / T[P[b]];
  std::vector<int32_t> tile(4 * nt, -1);
  acat::batch_tiles(np, n.data(), P.data(), T, tile.data(), first.data(), count.data());
  for (int64_t i = 0; i < nt; ++i) std::printf("%d %d %d %d\n", tile[4 * i], tile[4 * i + 1], tile[4 * i + 2], tile[4 * i + 3]);
  for (int b = 0; b < np; ++b) std::printf("%d %d\n", first[b], count[b]);
  return 0;
}
