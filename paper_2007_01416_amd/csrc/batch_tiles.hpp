// The tiles of a batch (host side): whether a step goes by tiles, and which cells each
// block of the tile launch steps.
#pragma once

#include <algorithm>
#include <cstdint>

#include "acat_internal.hpp"

namespace acat {

// How a batch is cut into tiles, and whether it is stepped by them.
struct BatchSplit {
  int T[BATCH_PMAX + 1];   // cells per tile of the problems of half-width P
  int64_t ntiles;
  bool by_tiles;
};

// T: 4 GPW r - 1 (r rounds of order P for each of a block's four waves, as in a
// single problem), r as large as leaves the batch some 4096 tiles, four times what
// the chip holds at once, so that the tiles dealt out last fill its gaps; and no
// smaller than holds the mean problem of that P whole, where that fits and those
// problems fill the chip by themselves (3000 Euler problems of 64 cells, P = 4, in
// three tiles each 121 us per step, in one 94).
//
// by_tiles: not where many problems fill little of their one tile each.  A tile then
// costs about what 100 interfaces (a scalar law: 80) cost in passes, which pack those
// of all problems into full blocks, but take five launches more, worth some 350000
// interfaces (480000); a full tile saves at least a tenth.  Steps of equal problems,
// tiles / passes, P = 1 and P = 4: Euler 40000 of 8 cells 212 us / 51 and 367 / 121, of
// 64 233 / 171 and 1010 / 928; 10000 of 64 62 / 59 and 272 / 258; 20000 of 100 126 / 140
// and 719 / 742; 5000 of 48 33 / 37 and 117 / 119; 3000 of 8 23 / 24 and 38 / 48.
// Burgers 40000 of 64 129 / 102 and 314 / 303, 10000 of 32 34 / 33 and 56 / 59, of 48
// 34 / 39 and 68 / 79.
// Never where the tiles' threads pass what a launch may hold (2^32).
inline BatchSplit batch_split(int nprob, const int64_t* n, const int32_t* P, int nvar) {
  BatchSplit s{};
  int64_t count[BATCH_PMAX + 1] = {}, cells[BATCH_PMAX + 1] = {}, ncell = 0;
  for (int b = 0; b < nprob; ++b) {
    ++count[P[b]];
    cells[P[b]] += n[b];
  }
  for (int p = 1; p <= BATCH_PMAX; ++p) ncell += cells[p];
  for (int p = 1; p <= BATCH_PMAX; ++p) {
    const int per = 4 * (p == 3 ? 10 : 32 / p), rmax = BLOCK / per;
    int64_t r = ncell / ((int64_t)per * 4096);
    if (count[p] >= 1024 && cells[p] < count[p] * BLOCK) r = std::max(r, cells[p] / count[p] / per + 1);
    s.T[p] = per * (int)(r < 1 ? 1 : r > rmax ? rmax : r) - 1;
  }
  int64_t idle = 0;
  const int64_t worth = nvar == 1 ? 80 : 100;
  for (int b = 0; b < nprob; ++b) {
    const int64_t t = (int64_t)((double)(n[b] + s.T[P[b]] - 1) / s.T[P[b]]);   // exact: both below 2^32
    s.ntiles += t;
    idle += n[b] < worth * t ? worth * t - n[b] : -(n[b] / 8);
  }
  s.by_tiles = idle <= (nvar == 1 ? 480000 : 350000) && s.ntiles < ((int64_t)1 << 32) / BLOCK;
  return s;
}

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
