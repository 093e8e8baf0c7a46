// The 1D step by tiles: one launch for a given time step, two for a CFL step
// (the wave-speed maxima, then the tiles), instead of one launch per pass and
// order class.  Where decisions are recorded or given, the tiles also write the
// class map and their interfaces per order, which one more launch adds up to the
// class counts (a single tile writes those itself): three launches where a
// launch per pass and class took P + 4 (Euler 20011 cells P = 3, a recorded step,
// a replayed one and the adjoint: 98 -> 53 us with the adjoint by tiles too).
#include <hip/hip_runtime.h>

#include "acat_internal.hpp"
#include "coeffs.hpp"
#include "step_common.hpp"
#include "tile1d.hpp"

namespace acat {
namespace {

#define ACAT_CHECK_LAUNCH()                  \
  do {                                       \
    hipError_t e_ = hipGetLastError();       \
    if (e_ != hipSuccess) return e_;         \
  } while (0)

// part[block] = the largest spectral radius of the block's cells;
// part[gridDim.x] = the time before the step (the tiles advance it).
constexpr int MAX_PARTS = 1024;
template <int FLUX, int NV>
__global__ __launch_bounds__(BLOCK) void k_speed1d(KProb pb, const double* __restrict__ u, double* part,
                                                   const double* t_dev) {
  __shared__ double red[NWAVE];
  double m = 0.0;
  for (int64_t e = (int64_t)blockIdx.x * BLOCK + threadIdx.x; e < pb.nx; e += (int64_t)gridDim.x * BLOCK) {
    double w[NV];
#pragma unroll
    for (int c = 0; c < NV; ++c) w[c] = u[c * pb.nx + e];
    m = fmax(m, spectral_radius<FLUX, 1, NV>(pb.ph, w, 0));
  }
  m = block_max(m, red);
  if (threadIdx.x == 0) {
    part[blockIdx.x] = m;
    if (blockIdx.x == 0) part[gridDim.x] = t_dev ? *t_dev : 0.0;
  }
}

// Tiles of T cells.  CFL mode: from nparts partial maxima, or, with nparts =
// 0, from the one tile that holds the whole problem.
// Four waves per SIMD up to P = 5 (bounded to 128 registers there, 137
// unbounded: 3e5 cells 218 -> 206 us per step), three at P = 6 (159).
template <int FLUX, int NV, int P, bool DEC>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(P <= 5 ? 4 : 3))) void k_tile1d(
    KProb pb, KStep st, int T, int nparts) {
  __shared__ TileMem<FLUX, NV, P> m;
  constexpr int G = TileMem<FLUX, NV, P>::G;
  const Tile t{st.u, st.uout, pb.nx, pb.nx, (int64_t)blockIdx.x * T, T, P, pb.bc, pb.dx};
  tile_load<FLUX, NV, P>(m, t);
  double dt;
  if (st.cfl_mode) {
    double s = 0.0, t0 = 0.0;
    if (nparts == 0) {
      if (st.t_dev) t0 = *st.t_dev;
      __syncthreads();
      if (threadIdx.x < pb.nx) {
        double uc[NV];
#pragma unroll
        for (int c = 0; c < NV; ++c) uc[c] = m.u[c][threadIdx.x + G];
        s = spectral_radius<FLUX, 1, NV>(pb.ph, uc, 0);
      }
    } else {
      for (int i = threadIdx.x; i < nparts; i += BLOCK) s = fmax(s, st.part[i]);
      t0 = st.part[nparts];
    }
    s = block_max(fmax(s, 0.0), m.red);
    dt = st.cfl * pb.dx / s;
    if (st.t_dev) dt = clip_dt(dt, t0, st.t_final);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      if (st.t_dev) *st.t_dev = t0 + dt;
      *st.dt_out = dt;
    }
  } else {
    dt = step_dt(st);
    __syncthreads();
  }
  double w[NV];
  const TileDec dec{st.ordx, st.psix, st.alx, st.cls, gridDim.x == 1 ? st.counts : st.list, st.replay != 0};
  tile_step<FLUX, NV, P, false, DEC>(m, t, pb.ph, pb.flags, pb.eps, pb.theta, dt, st.status, w, dec);
}

// counts[c] = the sum of class c over the tiles; one block per class
__global__ __launch_bounds__(BLOCK) void k_sum_counts(const int32_t* tiles, int ntiles, int32_t* counts) {
  __shared__ int ws[NWAVE];
  int n = 0;
  for (int i = threadIdx.x; i < ntiles; i += BLOCK) n += tiles[(int64_t)blockIdx.x * ntiles + i];
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) n += __shfl_xor(n, off);
  if (__lane_id() == 0) ws[threadIdx.x >> 6] = n;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < NWAVE; ++w) n += ws[w];
    counts[blockIdx.x] = n;
  }
}

template <int FLUX, int NV, int P, bool DEC>
hipError_t tile1d_impl(const KProb& pb, const KStep& st, hipStream_t s) {
  auto kern = k_tile1d<FLUX, NV, P, DEC>;
  static const int per_cu = [&] {
    int b = 0;
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, kern, BLOCK, 0) == hipSuccess && b > 0 ? b : 1;
  }();
  int T = tile_cells<P>(pb.nx, (int64_t)per_cu * num_cus(), 1, BLOCK), nparts = 0;
  if (st.cfl_mode) {
    // a problem of up to four rounds per wave in one block: the block reduces
    // the wave speeds itself (one launch)
    constexpr int GPW = Groups<2 * P, 64>::PER_BLOCK;
    if (pb.nx < BLOCK && pb.nx + 1 <= 4 * NWAVE * GPW) {
      T = (int)pb.nx;
    } else {
      nparts = (int)std::min<int64_t>((pb.nx + BLOCK - 1) / BLOCK, MAX_PARTS);
      ProfScope ps("speed1d", s);
      k_speed1d<FLUX, NV><<<nparts, BLOCK, 0, s>>>(pb, st.u, st.part, st.t_dev);
      ACAT_CHECK_LAUNCH();
    }
  }
  const int64_t nb = (pb.nx + T - 1) / T;
  // the tiles' counts, P for each, lie where a 2D step has its item lists, at least
  // nx entries: with T >= 2 P and nx >= 2 P, P ceil(nx / T) <= nx (one tile: P <= nx;
  // more: nx > T, and P (nx / T + 1) <= nx as (T + 1)(T - P) >= P T)
  static_assert(NWAVE * Groups<2 * P, 64>::PER_BLOCK - 1 >= 2 * P, "the tiles' counts fit the list");
  {
    ProfScope ps("step1d", s);
    kern<<<(unsigned)nb, BLOCK, 0, s>>>(pb, st, T, nparts);
  }
  ACAT_CHECK_LAUNCH();
  if (DEC && nb > 1) {
    ProfScope ps("class_counts", s);
    k_sum_counts<<<P, BLOCK, 0, s>>>(st.list, (int)nb, st.counts);
    ACAT_CHECK_LAUNCH();
  }
  return hipSuccess;
}

template <int FLUX, int NV, int P>
hipError_t tile1d_mode(const KProb& pb, const KStep& st, hipStream_t s) {
  return st.replay || st.recorded ? tile1d_impl<FLUX, NV, P, true>(pb, st, s)
                                  : tile1d_impl<FLUX, NV, P, false>(pb, st, s);
}

}  // namespace

hipError_t launch_step_1d(const KProb& pb, const KStep& st, hipStream_t s) {
  if (pb.flux == EUL) {
    switch (pb.P) {
      case 1: return tile1d_mode<EUL, 3, 1>(pb, st, s);
      case 2: return tile1d_mode<EUL, 3, 2>(pb, st, s);
      case 3: return tile1d_mode<EUL, 3, 3>(pb, st, s);
      case 4: return tile1d_mode<EUL, 3, 4>(pb, st, s);
      case 5: return tile1d_mode<EUL, 3, 5>(pb, st, s);
      case 6: return tile1d_mode<EUL, 3, 6>(pb, st, s);
    }
  } else if (pb.flux == BURG) {
    switch (pb.P) {
      case 1: return tile1d_mode<BURG, 1, 1>(pb, st, s);
      case 2: return tile1d_mode<BURG, 1, 2>(pb, st, s);
      case 3: return tile1d_mode<BURG, 1, 3>(pb, st, s);
      case 4: return tile1d_mode<BURG, 1, 4>(pb, st, s);
      case 5: return tile1d_mode<BURG, 1, 5>(pb, st, s);
      case 6: return tile1d_mode<BURG, 1, 6>(pb, st, s);
    }
  } else {
    switch (pb.P) {
      case 1: return tile1d_mode<ADV, 1, 1>(pb, st, s);
      case 2: return tile1d_mode<ADV, 1, 2>(pb, st, s);
      case 3: return tile1d_mode<ADV, 1, 3>(pb, st, s);
      case 4: return tile1d_mode<ADV, 1, 4>(pb, st, s);
      case 5: return tile1d_mode<ADV, 1, 5>(pb, st, s);
      case 6: return tile1d_mode<ADV, 1, 6>(pb, st, s);
    }
  }
  return hipErrorInvalidValue;
}

}  // namespace acat
