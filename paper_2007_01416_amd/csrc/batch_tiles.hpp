// The tiles of a batch (host side): which cells each block of the tile launch steps.
#pragma once

#include <cstdint>

#include "acat_internal.hpp"

namespace acat {

// tile[4 i .. 4 i + 3]: problem, first cell, cells per tile and slot of block i's
// tile, for tiles of T[P] cells; the slots of problem b are tfirst[b] ..
// tfirst[b] + tcount[b] - 1.  The blocks take the highest P first, its full tiles and
// then the remainders, the longest first, so that the launch ends on short ones and
// neighbouring blocks have tiles alike.  Blocks go to the XCDs in turn: with every
// problem's tiles side by side, one full and one remainder each, half the XCDs got
// all the full ones (1e4 problems of 256 cells, P = 3: 678 us per step, so 417; of
// 300 cells 658 and 468).
inline void batch_tiles(int nprob, const int64_t* n, const int32_t* P, const int* T, int32_t* tile, int32_t* tfirst,
                        int32_t* tcount) {
  int64_t at = 0, slot = 0;
  auto put = [&](int64_t i, int b, int64_t c0, int64_t s) {
    tile[4 * i] = b;
    tile[4 * i + 1] = (int32_t)c0;
    tile[4 * i + 2] = T[P[b]];
    tile[4 * i + 3] = (int32_t)s;
  };
  for (int q = BATCH_PMAX; q >= 1; --q) {
    int64_t of[BLOCK] = {};   // remainders of each length, then where the next one goes
    for (int b = 0; b < nprob; ++b) {
      if (P[b] != q) continue;
      const int64_t full = n[b] / T[q], rest = n[b] % T[q];
      tfirst[b] = (int32_t)slot;
      tcount[b] = (int32_t)(full + (rest > 0));
      for (int64_t k = 0; k < full; ++k) put(at++, b, k * T[q], slot + k);
      of[rest] += rest > 0;
      slot += tcount[b];
    }
    for (int r = BLOCK - 1; r >= 1; --r) {
      const int64_t c = of[r];
      of[r] = at;
      at += c;
    }
    for (int b = 0; b < nprob; ++b) {
      if (P[b] != q) continue;
      const int64_t full = n[b] / T[q], rest = n[b] % T[q];
      if (rest > 0) put(of[rest]++, b, full * T[q], tfirst[b] + full);
    }
  }
}

}  // namespace acat
