// One step of a tile of 1D cells by one block, from the states to the updated
// states, with nothing in memory between: the tile's cells and their stencil
// halo are staged in LDS, its interfaces classified, grouped by order in LDS,
// their fluxes computed wave by wave and the cells updated.  A tile of T
// cells has T + 1 interfaces; the one it shares with the next tile is
// computed by both, with the same operations on the same states.
//
// Against one launch per pass (classification, list prefix, list scatter, one
// flux launch per order, update) this leaves out the launches and the traffic
// of the class maps, lists, weights and interface fluxes.  What remains is
// bound by the fluxes' FP64 issue and dependency latency.  Measured per step,
// pass by pass -> by tiles: 200 cells P = 2 25.5 -> 8.9 us (eager), 4096
// cells P = 4 30.1 -> 14.7 us (graph), 4.2 M cells P = 6 3929 -> 3608 us, a
// batch of 256 problems of 1.2 M cells, P = 2..4, 325 -> 209 us.
#pragma once

#include <hip/hip_runtime.h>

#include "cat1d.hpp"
#include "step_common.hpp"

namespace acat {
namespace {

// doubles of LDS one wave's exchange takes, the largest over the orders 1..PM
template <int FLUX, int NV, int PM>
constexpr int wave_xs_doubles() {
  int m = Cat1D<FLUX, NV, 1, 64>::LDS_DOUBLES;
  if constexpr (PM >= 2) m = m > Cat1D<FLUX, NV, 2, 64>::LDS_DOUBLES ? m : Cat1D<FLUX, NV, 2, 64>::LDS_DOUBLES;
  if constexpr (PM >= 3) m = m > Cat1D<FLUX, NV, 3, 64>::LDS_DOUBLES ? m : Cat1D<FLUX, NV, 3, 64>::LDS_DOUBLES;
  if constexpr (PM >= 4) m = m > Cat1D<FLUX, NV, 4, 64>::LDS_DOUBLES ? m : Cat1D<FLUX, NV, 4, 64>::LDS_DOUBLES;
  if constexpr (PM >= 5) m = m > Cat1D<FLUX, NV, 5, 64>::LDS_DOUBLES ? m : Cat1D<FLUX, NV, 5, 64>::LDS_DOUBLES;
  if constexpr (PM >= 6) m = m > Cat1D<FLUX, NV, 6, 64>::LDS_DOUBLES ? m : Cat1D<FLUX, NV, 6, 64>::LDS_DOUBLES;
  return m;
}

template <int FLUX, int NV, int PM>
struct TileMem {
  static constexpr int G = PM > 2 ? PM : 2;
  static constexpr int NC = BLOCK - 1 + 2 * G;   // cells of the longest tile and its halo
  double u[NV][NC];
  double F[NV][BLOCK];
  double psi[BLOCK], al[BLOCK];                  // of the interfaces of order 1
  double xs[NWAVE][wave_xs_doubles<FLUX, NV, PM>()];
  double red[NWAVE];
  int wc[PM][NWAVE];                             // interfaces of each order per wave of the classification
  uint8_t list[BLOCK];                           // interfaces by order, the highest first
};

// The cells a tile steps: cells c0 .. c0 + T - 1 (those below n) of a problem
// whose component c starts at u + c * stride.
struct Tile {
  const double* u;
  double* uout;
  int64_t stride, n, c0;
  int T, P, bc;
  double dx;
};

// The decisions of a tile's interfaces: given (replay), or chosen and written; the
// class map and the tile's interfaces per order, counts[(p - 1) ntiles + tile],
// written in both.
struct TileDec {
  int8_t* ord;
  double* psi;
  double* al;
  int8_t* cls;
  int32_t* counts;
  bool replay;
};

// Stages cells c0 - G .. c0 + T + G - 1 through the boundary map, as far as
// the problem's last interface reads (n >= 2 G, so one wrap suffices); the
// caller's barrier follows.
template <int FLUX, int NV, int PM>
__device__ __forceinline__ void tile_load(TileMem<FLUX, NV, PM>& m, const Tile& t) {
  constexpr int G = TileMem<FLUX, NV, PM>::G;
  for (int j = threadIdx.x; j < t.T + 2 * G; j += BLOCK) {
    const int64_t x = t.c0 - G + j;
    if (x >= t.n + G) break;
    const int64_t s = bc_index(x, t.n, t.bc);
#pragma unroll
    for (int c = 0; c < NV; ++c) m.u[c][j] = t.u[c * t.stride + s];
  }
}

// Maximum of m over the block (every thread gets it); m >= 0 or NaN, which
// fmax drops.
__device__ __forceinline__ double block_max(double m, double* red) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) m = fmax(m, __shfl_xor(m, off));
  if (__lane_id() == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < NWAVE; ++w) m = fmax(m, red[w]);
  return m;
}

// One interface order of the tile: the wave's share of its rounds.  `task`
// runs over the rounds of all orders, the highest order first, dealt to the
// waves in turn.
template <int FLUX, int NV, int PM, int p>
__device__ __forceinline__ void tile_order(TileMem<FLUX, NV, PM>& m, const Phys& ph, int flags, double lam, double alf,
                                           double* xs, int first, int count, int& task) {
  using Cat = Cat1D<FLUX, NV, p, 64>;
  constexpr int G = TileMem<FLUX, NV, PM>::G;
  const int rounds = (count + Cat::PER_ROUND - 1) / Cat::PER_ROUND;
  if (task < rounds) {
    const Cat cat(__lane_id());
    for (; task < rounds; task += NWAVE) {
      const int it = task * Cat::PER_ROUND + cat.g;
      const bool valid = cat.in && it < count;
      const int k = valid ? m.list[first + it] : 0;
      double u[NV];
#pragma unroll
      for (int c = 0; c < NV; ++c) u[c] = valid ? m.u[c][k + G - p + cat.a] : 1.0;
      double Fc[2];
      cat.flux(ph, u, lam, xs, Fc[0], Fc[1]);
      if (!valid) continue;
#pragma unroll
      for (int s = 0; s < (NV > Cat::L ? 2 : 1); ++s) {
        const int c = cat.a + s * Cat::L;
        if (c >= NV) continue;
        double F = Fc[s];
        if constexpr (p == 1) {
          double uL[NV], uR[NV];
#pragma unroll
          for (int cc = 0; cc < NV; ++cc) {
            uL[cc] = m.u[cc][k + G - 1];
            uR[cc] = m.u[cc][k + G];
          }
          F = fl_cat2<FLUX, NV>(ph, flags, uL, uR, c, F, m.psi[k], m.al[k], alf);
        }
        m.F[c][k] = F;
      }
    }
  }
  task -= rounds;
}

// Classifies, computes the fluxes and updates a staged tile (after the
// barrier that follows tile_load).  RT: the largest half-width is t.P <= PM
// (run time), else PM.  w: the new state of cell threadIdx.x of the tile;
// returns whether the thread has one.  DEC: with the decisions of dec.
template <int FLUX, int NV, int PM, bool RT, bool DEC = false>
__device__ __forceinline__ bool tile_step(TileMem<FLUX, NV, PM>& m, const Tile& t, const Phys& ph, int flags,
                                          double eps, double theta, double dt, uint32_t* status, double (&w)[NV],
                                          const TileDec& dec = {}) {
  constexpr int G = TileMem<FLUX, NV, PM>::G;
  const int tid = threadIdx.x, lane = __lane_id(), wid = tid >> 6;
  const double lam = dt / t.dx;
  // interface k: between cells c0 - 1 + k and c0 + k
  const bool valid = tid <= t.T && t.c0 + tid <= t.n;
  int ps = 0;
  // the tile that holds the interface's left cell writes its decisions (the
  // first tile also those of a boundary interface to the left of all cells)
  [[maybe_unused]] const bool own = valid && (tid >= 1 || (t.c0 == 0 && t.bc != PERIODIC));
  [[maybe_unused]] const int64_t x = t.bc == PERIODIC ? (t.c0 + tid == 0 ? t.n : t.c0 + tid) - 1 : t.c0 + tid;
  if (DEC && dec.replay) {
    if (valid) {
      ps = dec.ord[x];
      if (ps < 1 || ps > PM) {   // invalid recorded order: taken as 1, flagged
        ps = 1;
        if (own) atomicOr(status, 4u);
      }
      if (ps == 1) {
        m.psi[tid] = dec.psi[x];
        m.al[tid] = dec.al[x];
      }
    }
  } else if (valid) {
    double v[NV][2 * G];
#pragma unroll
    for (int a = 0; a < 2 * G; ++a)
#pragma unroll
      for (int c = 0; c < NV; ++c) v[c][a] = m.u[c][tid + a];
    if constexpr (RT) ps = SelectRT<NV, G, PM>::run(v, t.P, eps, theta);
    else ps = Select<NV, G, PM>::run(v, eps, theta, (flags & FLAG_PSI2_MODIFIED) != 0);
    double psi = -1.0, al = -1.0;
    if (ps == 1) {
      low_order_weights<FLUX, NV, G>(ph, flags, v, psi, al);
      m.psi[tid] = psi;
      m.al[tid] = al;
    }
    if (DEC && own) {
      dec.ord[x] = (int8_t)ps;
      dec.psi[x] = psi;
      dec.al[x] = al;
    }
  }
  if (DEC && own) dec.cls[x] = (int8_t)(ps - 1);
  unsigned long long mine = 0ull;
#pragma unroll
  for (int p = 1; p <= PM; ++p) {
    const unsigned long long b = __ballot(ps == p);
    if (ps == p) mine = b;
    if (lane == 0) m.wc[p - 1][wid] = __popcll(b);
  }
  __syncthreads();
  int count[PM + 1], first[PM + 1], run = 0;
#pragma unroll
  for (int p = PM; p >= 1; --p) {
    first[p] = run;
    int pos = run;
    count[p] = 0;
#pragma unroll
    for (int q = 0; q < NWAVE; ++q) {
      const int n = __builtin_amdgcn_readfirstlane(m.wc[p - 1][q]);
      if (q < wid) pos += n;
      count[p] += n;
    }
    if (ps == p) m.list[pos + __popcll(mine & ((1ull << lane) - 1ull))] = (uint8_t)tid;
    run += count[p];
  }
  if (DEC && tid == 0) {
#pragma unroll
    for (int p = 1; p <= PM; ++p)
      dec.counts[(p - 1) * (int64_t)gridDim.x + blockIdx.x] = count[p] - (ps == p && !own ? 1 : 0);
  }
  __syncthreads();
  const double alf = t.dx / dt;
  int task = __builtin_amdgcn_readfirstlane(wid);
  double* xs = m.xs[wid];
  if constexpr (PM >= 6) tile_order<FLUX, NV, PM, 6>(m, ph, flags, lam, alf, xs, first[6], count[6], task);
  if constexpr (PM >= 5) tile_order<FLUX, NV, PM, 5>(m, ph, flags, lam, alf, xs, first[5], count[5], task);
  if constexpr (PM >= 4) tile_order<FLUX, NV, PM, 4>(m, ph, flags, lam, alf, xs, first[4], count[4], task);
  if constexpr (PM >= 3) tile_order<FLUX, NV, PM, 3>(m, ph, flags, lam, alf, xs, first[3], count[3], task);
  if constexpr (PM >= 2) tile_order<FLUX, NV, PM, 2>(m, ph, flags, lam, alf, xs, first[2], count[2], task);
  tile_order<FLUX, NV, PM, 1>(m, ph, flags, lam, alf, xs, first[1], count[1], task);
  __syncthreads();
  if (tid >= t.T || t.c0 + tid >= t.n) return false;
  bool finite = true;
#pragma unroll
  for (int c = 0; c < NV; ++c) {
    w[c] = m.u[c][tid + G] + lam * (m.F[c][tid] - m.F[c][tid + 1]);
    t.uout[c * t.stride + t.c0 + tid] = w[c];
    finite = finite && isfinite(w[c]);
  }
  const uint32_t bad = (finite ? 0u : 1u) | (physical<FLUX, 1, NV>(ph, w) ? 0u : 2u);
  if (bad) atomicOr(status, bad);
  return true;
}

}  // namespace
}  // namespace acat
