// Batched ACAT step: many independent 1D problems (own size N_b, largest
// half-width P_b, boundary, dx_b and time step dt_b; common flux) advanced
// together.  The interfaces of all problems are classified in one launch,
// grouped into per-order work lists shared by all problems, and each order
// class is one persistent launch over every problem, so the small problems
// of a batch fill the GPU together.  That is the path of a batch with a launch
// table, or of very many very small problems; else the whole step is one launch
// over tiles of the problems (tile1d.hpp; the line: batch_split).  Per interface the arithmetic is that of the single-problem
// kernels (same rounding), so a batched step equals the per-problem steps bit
// for bit.
//
// Layout: states are SoA over the concatenated cells, u[var][coff_b + i];
// interface arrays are concatenated the same way with offsets ioff_b.
#include <hip/hip_runtime.h>

#include "acat_internal.hpp"
#include "cat1d.hpp"
#include "coeffs.hpp"
#include "step_common.hpp"
#include "tile1d.hpp"

namespace acat {

namespace {

constexpr int GW = BATCH_PMAX;   // indicator window half-width for every problem (offsets -3 .. 4)

template <int FLUX, int NV>
__global__ __launch_bounds__(BLOCK) void k_classify_b(KBatch bt, KBStep st) {
  const int64_t kg = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  const bool valid = kg < bt.nif;
  int ps = 1;
  if (valid) {
    const int b = bt.pif[kg];
    const int n = bt.N[b], bc = bt.bc[b];
    const int i = (int)(kg - bt.ioffs[b]) - (bc == PERIODIC ? 0 : 1);
    const double* ub = st.u + bt.coff[b];
    double v[NV][2 * GW];
#pragma unroll
    for (int a = 0; a < 2 * GW; ++a) {
      const int node = bc_index32(i - GW + 1 + a, n, bc);
#pragma unroll
      for (int c = 0; c < NV; ++c) v[c][a] = ub[c * bt.ncell + node];
    }
    ps = SelectRT<NV, GW, BATCH_PMAX>::run(v, bt.P[b], bt.eps, bt.theta);
    double psi1 = -1.0, al = -1.0;
    if (ps == 1) low_order_weights<FLUX, NV, GW>(bt.ph, 0, v, psi1, al);
    st.ord[kg] = (int8_t)ps;
    st.psi[kg] = psi1;
    st.al[kg] = al;
  }
  __shared__ int sh[MAX_CLASSES];
  block_hist(sh, valid, ps - 1, st.hist);
}

// Interfaces of order p of every problem, BS threads per block; xs: LDS, LDS_DOUBLES.
template <int FLUX, int NV, int p, int BS>
__device__ __forceinline__ void flux_b_body(const KBatch& bt, const KBStep& st, double* xs) {
  using Cat = Cat1D<FLUX, NV, p, BS>;
  const Cat cat(threadIdx.x);
  const Slice sl(st.counts, st.list, p - 1, Cat::PER_ROUND);
  for (int64_t base = sl.lo; base < sl.hi; base += Cat::PER_ROUND) {
    const bool valid = cat.in && base + cat.g < sl.hi;
    const int64_t kg = valid ? sl.items[base + cat.g] : 0;
    const int b = bt.pif[kg];
    const int n = bt.N[b], bc = bt.bc[b];
    const int i = (int)(kg - bt.ioffs[b]) - (bc == PERIODIC ? 0 : 1);
    const double* ub = st.u + bt.coff[b];
    const double lam = st.dt[b] / bt.dx[b];
    const int node = bc_index32(i + (cat.a - p + 1), n, bc);
    double u[NV];
#pragma unroll
    for (int c = 0; c < NV; ++c) u[c] = valid ? ub[c * bt.ncell + node] : 1.0;
    double Fc[2];
    cat.flux(bt.ph, u, lam, xs, Fc[0], Fc[1]);
    if (!valid) continue;
#pragma unroll
    for (int task = 0; task < (NV > Cat::L ? 2 : 1); ++task) {
      const int c = cat.a + task * Cat::L;
      if (c >= NV) continue;
      double F = Fc[task];
      if constexpr (p == 1) {
        const int nl = bc_index32(i, n, bc), nr = bc_index32(i + 1, n, bc);
        double uL[NV], uR[NV];
#pragma unroll
        for (int cc = 0; cc < NV; ++cc) {
          uL[cc] = ub[cc * bt.ncell + nl];
          uR[cc] = ub[cc * bt.ncell + nr];
        }
        F = fl_cat2<FLUX, NV>(bt.ph, 0, uL, uR, c, F, st.psi[kg], st.al[kg], 0.0);
      }
      st.F[c * bt.nif + kg] = F;
    }
  }
}

template <int FLUX, int NV, int p, int BS>
__global__ __launch_bounds__(BS) void k_flux_b(KBatch bt, KBStep st) {
  __shared__ double xs[Cat1D<FLUX, NV, p, BS>::LDS_DOUBLES];
  flux_b_body<FLUX, NV, p, BS>(bt, st, xs);
}

// The orders below PM in one launch (a batch without a launch table): every block
// runs its share of each list in turn.
template <int FLUX, int NV, int PM>
__global__ __launch_bounds__(BLOCK) void k_flux_low_b(KBatch bt, KBStep st) {
  constexpr int a = Cat1D<FLUX, NV, 1, BLOCK>::LDS_DOUBLES, b = Cat1D<FLUX, NV, 2, BLOCK>::LDS_DOUBLES;
  constexpr int c = Cat1D<FLUX, NV, 3, BLOCK>::LDS_DOUBLES;
  __shared__ double xs[a > b ? (a > c ? a : c) : (b > c ? b : c)];
  if constexpr (PM > 3) {
    flux_b_body<FLUX, NV, 3, BLOCK>(bt, st, xs);
    __syncthreads();
  }
  if constexpr (PM > 2) {
    flux_b_body<FLUX, NV, 2, BLOCK>(bt, st, xs);
    __syncthreads();
  }
  flux_b_body<FLUX, NV, 1, BLOCK>(bt, st, xs);
}

// A wave speed as a maximum candidate: NaN and -0 become +0, so that the bit
// pattern orders like the value under an unsigned integer maximum.
__device__ __forceinline__ double speed_floor(double m) { return m > 0.0 ? m : 0.0; }

template <int FLUX, int NV, bool CFL>
__global__ __launch_bounds__(BLOCK) void k_update_b(KBatch bt, KBStep st) {
  const int64_t e = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  const bool valid = e < bt.ncell;
  const int b = valid ? bt.pcell[e] : 0;
  double w[NV];
  if (valid) {
    const int n = bt.N[b], bc = bt.bc[b];
    const int i = (int)(e - bt.coff[b]);
    const double lam = st.dt[b] / bt.dx[b];
    const int64_t kr = bt.ioffs[b] + i + (bc == PERIODIC ? 0 : 1);
    const int64_t kl = bt.ioffs[b] + ((bc == PERIODIC) ? (i == 0 ? n - 1 : i - 1) : i);
    bool finite = true;
#pragma unroll
    for (int c = 0; c < NV; ++c) {
      w[c] = st.u[c * bt.ncell + e] + lam * (st.F[c * bt.nif + kl] - st.F[c * bt.nif + kr]);
      st.uout[c * bt.ncell + e] = w[c];
      finite = finite && isfinite(w[c]);
    }
    const uint32_t bad = (finite ? 0u : 1u) | (physical<FLUX, 1, NV>(bt.ph, w) ? 0u : 2u);
    if (bad) atomicOr(st.status, bad);
  }
  if constexpr (CFL) {
    // per-problem maximum of the new state's spectral radius (NaN and -0
    // count as +0, as in k_max_speed_b).  The lanes of a wave hold runs of
    // equal problem index: a segmented maximum over the runs, then the last
    // lane of each run stores it, with a plain store when the run is the
    // whole wave (most waves; folded per problem by k_dt_fold_b) and as an
    // atomic maximum on the bit patterns otherwise (only waves that straddle
    // problems; non-negative doubles order like their bit patterns, and max
    // is exact in any order).
    double m = valid ? speed_floor(spectral_radius<FLUX, 1, NV>(bt.ph, w, 0)) : 0.0;
    const int key = valid ? b : -1;
    const int lane = __lane_id();
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const double mo = __shfl_up(m, off);
      const int ko = __shfl_up(key, off);
      if (lane >= off && ko == key) m = fmax(m, mo);
    }
    const int key0 = __shfl(key, 0);
    const bool whole = __all(key == key0) && key0 >= 0;
    const int knext = __shfl_down(key, 1);
    if (valid && (lane == 63 || knext != key)) {
      if (whole) st.wmax[e >> 6] = m;
      else atomicMax(&st.smax[key], (unsigned long long)__double_as_longlong(m));
    }
  }
}

// The whole step of one tile of one problem per block; CFL: and the largest
// spectral radius of its new cells (NaN and -0 count as +0), in the tile's slot.
template <int FLUX, int NV, bool CFL>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(4))) void k_tile_b(KBatch bt, KBStep st) {
  __shared__ TileMem<FLUX, NV, BATCH_PMAX> m;
  const int32_t* tl = bt.tiles + 4 * (int64_t)blockIdx.x;
  const int b = tl[0];
  const int64_t off = bt.coff[b];
  const Tile t{st.u + off, st.uout + off, bt.ncell, bt.N[b], tl[1], tl[2], bt.P[b], bt.bc[b], bt.dx[b]};
  const double dt = st.dt[b];
  tile_load<FLUX, NV, BATCH_PMAX>(m, t);
  __syncthreads();
  double w[NV];
  const bool has = tile_step<FLUX, NV, BATCH_PMAX, true>(m, t, bt.ph, 0, bt.eps, bt.theta, dt, st.status, w);
  if constexpr (CFL) {
    const double s = block_max(has ? speed_floor(spectral_radius<FLUX, 1, NV>(bt.ph, w, 0)) : 0.0, m.red);
    if (threadIdx.x == 0) st.tmax[tl[3]] = s;
  }
}

// dt[b] = cfl dx[b] / (the largest of problem b's tiles), one wave per problem.
__global__ __launch_bounds__(64) void k_dt_tiles_b(KBatch bt, const double* tmax, double cfl, double* dt) {
  const int b = blockIdx.x;
  const double* mine = tmax + bt.tfirst[b];
  double m = 0.0;
  for (int i = threadIdx.x; i < bt.tcount[b]; i += 64) m = fmax(m, mine[i]);
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) m = fmax(m, __shfl_xor(m, off));
  if (threadIdx.x == 0) dt[b] = cfl * bt.dx[b] / m;
}

// smax[b] = max spectral radius over problem b: one 1024-thread block per
// problem (a few cells per thread even for the largest problems), no atomics.
constexpr int MSB_T = 1024;
template <int FLUX, int NV>
__global__ __launch_bounds__(MSB_T) void k_max_speed_b(KBatch bt, const double* __restrict__ u,
                                                      unsigned long long* smax) {
  const int b = blockIdx.x;
  const int64_t c0 = bt.coff[b], c1 = bt.coff[b + 1];
  double m = 0.0;
  for (int64_t e = c0 + threadIdx.x; e < c1; e += MSB_T) {
    double w[NV];
#pragma unroll
    for (int c = 0; c < NV; ++c) w[c] = u[c * bt.ncell + e];
    m = fmax(m, spectral_radius<FLUX, 1, NV>(bt.ph, w, 0));
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) m = fmax(m, __shfl_xor(m, off));
  __shared__ double red[MSB_T / 64];
  if (__lane_id() == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int w = 1; w < MSB_T / 64; ++w) m = fmax(m, red[w]);
    smax[b] = (unsigned long long)__double_as_longlong(speed_floor(m));
  }
}

// dt[b] = cfl dx[b] / smax[b]; smax is cleared for the next reduction
// One wave per problem: the maximum of the partial maxima of the waves whole
// inside problem b (cells coff[b] .. coff[b+1]-1) and of smax[b].
__global__ __launch_bounds__(64) void k_dt_fold_b(KBatch bt, unsigned long long* smax, const double* wmax,
                                                  double cfl, double* dt) {
  const int b = blockIdx.x;
  const int64_t w0 = (bt.coff[b] + 63) >> 6, w1 = bt.coff[b + 1] >> 6;
  double m = 0.0;
  for (int64_t v = w0 + threadIdx.x; v < w1; v += 64) m = fmax(m, wmax[v]);
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) m = fmax(m, __shfl_xor(m, off));
  if (threadIdx.x == 0) {
    m = fmax(m, __longlong_as_double((long long)smax[b]));
    dt[b] = cfl * bt.dx[b] / m;
    smax[b] = 0ull;
  }
}

__global__ void k_dt_b(KBatch bt, unsigned long long* smax, double cfl, double* dt) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b < bt.nprob) {
    dt[b] = cfl * bt.dx[b] / __longlong_as_double((long long)smax[b]);
    smax[b] = 0ull;
  }
}

#define ACAT_CHECK_LAUNCH()                  \
  do {                                       \
    hipError_t e_ = hipGetLastError();       \
    if (e_ != hipSuccess) return e_;         \
  } while (0)

template <int FLUX, int NV, int p, int BS>
hipError_t launch_flux_b_bs(const KBatch& bt, const KBStep& st, hipStream_t s) {
  static const char* names[5] = {"", "flux_b_p1", "flux_b_p2", "flux_b_p3", "flux_b_p4"};
  auto kern = k_flux_b<FLUX, NV, p, BS>;
  const int grid = persistent_grid(kern, bt.nif, 0, BS, bt.per_cu[p]);
  {
    ProfScope ps(names[p], s);
    kern<<<grid, BS, 0, s>>>(bt, st);
  }
  ACAT_CHECK_LAUNCH();
  return hipSuccess;
}

// launch shape of class p from the batch's tuning table (waves per block)
template <int FLUX, int NV, int p>
hipError_t launch_flux_b(const KBatch& bt, const KBStep& st, hipStream_t s) {
  if (p > bt.Pmax) return hipSuccess;
  switch (bt.waves[p]) {
    case 1: return launch_flux_b_bs<FLUX, NV, p, 64>(bt, st, s);
    case 2: return launch_flux_b_bs<FLUX, NV, p, 128>(bt, st, s);
    default: return launch_flux_b_bs<FLUX, NV, p, 256>(bt, st, s);
  }
}

// the highest order, then the others
template <int FLUX, int NV, int PM>
hipError_t launch_flux_two_b(const KBatch& bt, const KBStep& st, hipStream_t s) {
  const hipError_t e = launch_flux_b<FLUX, NV, PM>(bt, st, s);
  if (PM == 1 || e != hipSuccess) return e;
  if constexpr (PM > 1) {
    auto kern = k_flux_low_b<FLUX, NV, PM>;
    const int grid = persistent_grid(kern, bt.nif, 0);
    ProfScope ps("flux_b_low", s);
    kern<<<grid, BLOCK, 0, s>>>(bt, st);
  }
  ACAT_CHECK_LAUNCH();
  return hipSuccess;
}

template <int FLUX, int NV>
hipError_t tiles_b_impl(const KBatch& bt, const KBStep& st, hipStream_t s) {
  {
    ProfScope ps("step_b", s);
    if (st.smax) k_tile_b<FLUX, NV, true><<<bt.ntiles, BLOCK, 0, s>>>(bt, st);
    else k_tile_b<FLUX, NV, false><<<bt.ntiles, BLOCK, 0, s>>>(bt, st);
  }
  ACAT_CHECK_LAUNCH();
  if (st.smax) {
    k_dt_tiles_b<<<bt.nprob, 64, 0, s>>>(bt, st.tmax, st.cfl, st.dt_next);
    ACAT_CHECK_LAUNCH();
  }
  return hipSuccess;
}

template <int FLUX, int NV>
hipError_t step_b_impl(const KBatch& bt, const KBStep& st, hipStream_t s) {
  if (bt.by_tiles) return tiles_b_impl<FLUX, NV>(bt, st, s);
  const int cblocks = (int)((bt.nif + BLOCK - 1) / BLOCK);
  {
    ProfScope ps("classify_b", s);
    k_classify_b<FLUX, NV><<<cblocks, BLOCK, 0, s>>>(bt, st);
  }
  ACAT_CHECK_LAUNCH();
  k_scan_hist<<<bt.Pmax, SCAN_T, 0, s>>>(st.hist, cblocks, st.offs, st.counts, bt.Pmax, CflReduce{});
  ACAT_CHECK_LAUNCH();
  k_scatter<BATCH_PMAX, false><<<cblocks, BLOCK, 0, s>>>(st.ord, 1, bt.nif, 1, cblocks, st.offs, st.counts,
                                                         st.list);
  ACAT_CHECK_LAUNCH();
  hipError_t e = hipSuccess;
  if (bt.two_launches) {
    switch (bt.Pmax) {
      case 1: e = launch_flux_two_b<FLUX, NV, 1>(bt, st, s); break;
      case 2: e = launch_flux_two_b<FLUX, NV, 2>(bt, st, s); break;
      case 3: e = launch_flux_two_b<FLUX, NV, 3>(bt, st, s); break;
      default: e = launch_flux_two_b<FLUX, NV, 4>(bt, st, s); break;
    }
    if (e != hipSuccess) return e;
  } else {
    if ((e = launch_flux_b<FLUX, NV, 1>(bt, st, s)) != hipSuccess) return e;
    if ((e = launch_flux_b<FLUX, NV, 2>(bt, st, s)) != hipSuccess) return e;
    if ((e = launch_flux_b<FLUX, NV, 3>(bt, st, s)) != hipSuccess) return e;
    if ((e = launch_flux_b<FLUX, NV, 4>(bt, st, s)) != hipSuccess) return e;
  }
  {
    ProfScope ps("update_b", s);
    const unsigned grid = (unsigned)((bt.ncell + BLOCK - 1) / BLOCK);
    if (st.smax) k_update_b<FLUX, NV, true><<<grid, BLOCK, 0, s>>>(bt, st);
    else k_update_b<FLUX, NV, false><<<grid, BLOCK, 0, s>>>(bt, st);
  }
  ACAT_CHECK_LAUNCH();
  if (st.smax) {
    k_dt_fold_b<<<bt.nprob, 64, 0, s>>>(bt, st.smax, st.wmax, st.cfl, st.dt_next);
    ACAT_CHECK_LAUNCH();
  }
  return hipSuccess;
}

template <int FLUX, int NV>
hipError_t cfl_b_impl(const KBatch& bt, const double* u, double cfl, unsigned long long* smax, double* dt,
                      hipStream_t s) {
  {
    ProfScope ps("max_speed_b", s);
    k_max_speed_b<FLUX, NV><<<bt.nprob, MSB_T, 0, s>>>(bt, u, smax);
  }
  ACAT_CHECK_LAUNCH();
  k_dt_b<<<(bt.nprob + BLOCK - 1) / BLOCK, BLOCK, 0, s>>>(bt, smax, cfl, dt);
  ACAT_CHECK_LAUNCH();
  return hipSuccess;
}

}  // namespace

hipError_t launch_step_batched(const KBatch& bt, const KBStep& st, hipStream_t s) {
  if (bt.flux == EUL) return step_b_impl<EUL, 3>(bt, st, s);
  if (bt.flux == BURG) return step_b_impl<BURG, 1>(bt, st, s);
  return step_b_impl<ADV, 1>(bt, st, s);
}

hipError_t launch_cfl_batched(const KBatch& bt, const double* u, double cfl, unsigned long long* smax, double* dt,
                              hipStream_t s) {
  if (bt.flux == EUL) return cfl_b_impl<EUL, 3>(bt, u, cfl, smax, dt, s);
  if (bt.flux == BURG) return cfl_b_impl<BURG, 1>(bt, u, cfl, smax, dt, s);
  return cfl_b_impl<ADV, 1>(bt, u, cfl, smax, dt, s);
}

}  // namespace acat
