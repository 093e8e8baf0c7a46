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

// a launch of three classes (numbers 4, 0 and 2 of the lists, 7, 256 and 16
// items per round) with the given list lengths
long bad_items(const int (&n)[3], int nblk, std::mt19937& rng) {
  constexpr int cls[3] = {4, 0, 2}, per[3] = {7, 256, 16};
  std::vector<int32_t> counts(MAX_CLASSES, 0);
  for (int k = 0; k < 3; ++k) counts[cls[k]] = n[k];
  counts[1] = 5;   // a class of another launch
  int total = 0, first[MAX_CLASSES];
  for (int c = 0; c < MAX_CLASSES; ++c) {
    first[c] = total;
    total += counts[c];
  }
  std::vector<int32_t> list(total), taken(total, 0);
  std::vector<int32_t> tickets(MAX_CLASSES * NXCD * TICKET_STRIDE, 0);
  for (int i = 0; i < total; ++i) list[i] = i;
  KStep st{};
  st.counts = counts.data();
  st.list = list.data();
  st.tickets = tickets.data();
  std::vector<ChunkTable> tab(nblk);
  std::vector<Chunks<3>> blk;
  blk.reserve(nblk);
  for (int b = 0; b < nblk; ++b)
    blk.emplace_back(st, tab[b], 1, b, nblk, [&](int k, int& c, int& p) {
      c = cls[k];
      p = per[k];
    });
  long bad = 0;
  std::vector<int> live(nblk), at(nblk, -1);   // at: item the block's chunk has come to (-1: no chunk)
  for (int b = 0; b < nblk; ++b) live[b] = b;
  while (!live.empty()) {
    const size_t i = rng() % live.size();
    const int b = live[i];
    auto& c = blk[b];
    if (at[b] < 0) {
      if (!c.start(st, tab[b])) {
        live[i] = live.back();
        live.pop_back();
        continue;
      }
      at[b] = c.base;
    }
    for (int g = 0; g < per[c.cls]; ++g)
      if (at[b] + g < c.end) {
        const int item = c.items[at[b] + g];
        ++taken[item];
        bad += item < first[cls[c.cls]] || item >= first[cls[c.cls]] + n[c.cls];
      }
    at[b] += per[c.cls];
    if (at[b] >= c.end) {
      c.advance(tab[b]);
      at[b] = -1;
    }
  }
  for (int i = 0; i < total; ++i) bad += taken[i] != (i < first[1] || i >= first[1] + 5);
  return bad;
}

int main() {
  std::mt19937 rng(3);
  threadIdx = {0, 0, 0};
  long bad = 0, cases = 0;
  for (int nblk : {8, 16, 72, 768})
    for (int rounds : {0, 1, 2, 9, 15, 16, 63, 64, 130})
      for (int d : {-9, -1, 0, 1, 2, 13}) {
        const int a = rounds * 7 * nblk + d, b = (int)(rng() % 3) * 256 * nblk + d, c = (int)(rng() % (16 * nblk));
        if (a < 0 || b < 0 || (long)rounds * nblk > 20000) continue;
        const int lens[4][3] = {{a, b, c}, {a, 0, 0}, {0, b, 0}, {a, 1, c}};
        for (const auto& n : lens) bad += bad_items(n, nblk, rng);
        cases += 4;
      }
  std::printf("%ld %ld\n", bad, cases);
  return 0;
}
