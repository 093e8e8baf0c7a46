// The persistent blocks' shares of a class list (Chunks of step_common.hpp) on
// the CPU: the blocks of a launch take their rounds in an interleaved order,
// one thread standing for a block.  Prints the number of items not taken
// exactly once, over list lengths around whole rounds, shares and chunks.
#include "hip/hip_runtime.h"

#include <random>
#include <vector>

thread_local dim3s threadIdx, blockIdx;
dim3s gridDim, blockDim;
pthread_barrier_t g_block_barrier;
static int atomicAdd(int32_t* p, int v) {
  const int old = *p;
  *p += v;
  return old;
}
#define __syncthreads() ((void)0)
#define __builtin_amdgcn_readfirstlane(v) (v)
#include "step_common.hpp"

using namespace acat;

template <int PER_ROUND, bool PAIRED>
long bad_items(int n, int nblk, std::mt19937& rng) {
  const int cls = 2, before = 5;
  std::vector<int32_t> counts(MAX_CLASSES, 0), list(before + n), taken(before + n, 0);
  std::vector<int32_t> tickets(MAX_CLASSES * NXCD * TICKET_STRIDE, 0);
  counts[0] = before;
  counts[cls] = n;
  for (int i = 0; i < before + n; ++i) list[i] = i;
  KStep st{};
  st.counts = counts.data();
  st.list = list.data();
  st.tickets = tickets.data();
  std::vector<Chunks<PER_ROUND, PAIRED>> blk;
  std::vector<int32_t> sh(2 * nblk, 0);
  for (int b = 0; b < nblk; ++b) blk.emplace_back(st, cls, b, nblk);
  std::vector<int> live(nblk);
  for (int b = 0; b < nblk; ++b) live[b] = b;
  while (!live.empty()) {
    const size_t k = rng() % live.size();
    auto& c = blk[live[k]];
    if (c.base >= c.end) {
      live[k] = live.back();
      live.pop_back();
      continue;
    }
    for (int g = 0; g < PER_ROUND; ++g)
      if (c.base + g < c.end) ++taken[c.items[c.base + g]];
    c.advance(&sh[2 * live[k]]);
  }
  long bad = 0;
  for (int i = 0; i < before + n; ++i) bad += taken[i] != (i >= before);
  return bad;
}

int main() {
  std::mt19937 rng(3);
  threadIdx = {0, 0, 0};
  long bad = 0, cases = 0;
  for (int nblk : {8, 16, 72, 768})
    for (int rounds : {0, 1, 2, 11, 12, 15, 16, 63, 64, 200}) {
      if ((long)rounds * nblk > 20000) continue;
      for (int d : {-9, -1, 0, 1, 2, 13}) {
        const int n7 = rounds * 7 * nblk + d, n16 = rounds * 16 * nblk + d;
        if (n7 < 0) continue;
        bad += bad_items<7, false>(n7, nblk, rng) + bad_items<7, true>(n7, nblk, rng);
        bad += bad_items<16, false>(n16, nblk, rng) + bad_items<16, true>(n16, nblk, rng);
        cases += 4;
      }
    }
  std::printf("%ld %ld\n", bad, cases);
  return 0;
}
