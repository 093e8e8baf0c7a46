// ACAT 2D forward step on gfx950: classification, flux kernels over the order
// classes, conservative update; and the CFL reductions of 1D and 2D.
//
// Data flow of one step (all on one stream, no host synchronisation):
//   k_classify2d   one thread per corner: smoothness indicators psi^p
//                  (Sec. 3.2, minimum over components, Sec. 3.4), order p_s
//                  (Sec. 3, admissible set), and where p_s = 1 the superbee
//                  weight psi^1 (Sec. 3.1) and the Rusanov speed; writes the
//                  corner's order class as one byte, and a per-block histogram
//   k_scan_hist    large grids: per-class exclusive prefix of the tile
//                  histograms (and, in CFL mode, the time step from the
//                  classification's per-block maxima); small grids: a part
//                  of k_scatter
//   k_scatter      the item lists: every class's items in tile order
//                  (wave ballots, no global atomics)
//   k_flux2d       one or two persistent launches for all classes, whose blocks
//                  draw chunks of the class lists.  A list is processed in
//                  rounds, one LANE PER STENCIL NODE: a corner of orders
//                  (q1, q2) 2q1 x 2q2 lanes.  Each lane keeps its node's state
//                  and Taylor predictions in registers and evaluates the flux
//                  at its own predicted states; the spatial derivatives of the
//                  time-derivative fluxes go through LDS (Sec. 4 corner
//                  recursion)
//   k_update2d     conservative flux-difference update + status bits
#include <hip/hip_runtime.h>

#include <utility>

#include "acat_internal.hpp"
#include "coeffs.hpp"
#include "step_common.hpp"

namespace acat {
namespace {

__global__ void k_zero_u64(unsigned long long* p, int n) {
  const int t = threadIdx.x;
  if (t < n) p[t] = 0ull;
}

// ======================================================================= 2D
// One block per 16 x 16 tile of corners, one thread per corner.  The cells
// the tile's x- and y-stencils read (the tile and a halo of G - 1 below and
// G beyond it in each direction) are staged in LDS once per block.
template <int FLUX, int NV, int P>
__global__ __launch_bounds__(BLOCK) void k_classify2d(KProb pb, KStep st) {
  constexpr int G = P > 2 ? P : 2;
  constexpr int TW = TILE_X + 2 * G - 1, TH = TILE_Y + 2 * G - 1;
  static_assert(TILE_X * TILE_Y == BLOCK, "one thread per corner of the tile");
  __shared__ double tile[NV][TH][TW];
  const int64_t ntx = (pb.n1 + TILE_X - 1) / TILE_X;
  const int tx = threadIdx.x % TILE_X, ty = threadIdx.x / TILE_X;
  const int64_t e1 = (blockIdx.x % ntx) * TILE_X + tx;
  const int64_t e2 = (blockIdx.x / ntx) * TILE_Y + ty;
  const bool inside = e1 < pb.n1 && e2 < pb.n2;
  const int64_t e = e2 * pb.n1 + e1;
  const int64_t nx = pb.nx, ny = pb.ny;
  const int64_t i1 = inside ? e1 + pb.ioff : 0;
  const int64_t i2 = inside ? e2 + pb.ioff : 0;
  const bool needF = i2 >= 0, needG = i1 >= 0;
  const bool valid = inside && (needF || needG);
  if (!st.replay) {
    // tile cell (a, b) is cell (Y0 + a, X0 + b) before the boundary mapping;
    // cells beyond what the grid's last corner reads are not loaded (so the
    // periodic wrap stays within one period)
    const int64_t X0 = (blockIdx.x % ntx) * TILE_X + pb.ioff - G + 1;
    const int64_t Y0 = (blockIdx.x / ntx) * TILE_Y + pb.ioff - G + 1;
    const int64_t Xmax = pb.n1 - 1 + pb.ioff + G, Ymax = pb.n2 - 1 + pb.ioff + G;
    for (int t = threadIdx.x; t < TH * TW; t += BLOCK) {
      const int a = t / TW, b = t - a * TW;
      if (X0 + b <= Xmax && Y0 + a <= Ymax) {
        const int64_t x = bc_index(X0 + b, nx, pb.bc), y = bc_index(Y0 + a, ny, pb.bc);
#pragma unroll
        for (int c = 0; c < NV; ++c) tile[c][a][b] = st.u[(c * ny + y) * nx + x];
      }
    }
    __syncthreads();
  }
  int q1 = 1, q2 = 1;
  double sx = 0.0, sy = 0.0;
  if (valid) {
    const int64_t r2 = bc_index(i2, ny, pb.bc);   // ghost rows read the clamped row
    const int64_t r1 = bc_index(i1, nx, pb.bc);
    if (st.replay) {
      q1 = st.ordx[r2 * pb.nIx + (i1 - pb.ioff)];
      q2 = st.ordy[(i2 - pb.ioff) * nx + r1];
      if (q1 < 1 || q1 > P || q2 < 1 || q2 > P) {   // invalid recorded order: fall back to 1, flag it
        q1 = (q1 < 1 || q1 > P) ? 1 : q1;
        q2 = (q2 < 1 || q2 > P) ? 1 : q2;
        atomicOr(st.status, 4u);
      }
    } else {
      double v[NV][2 * G];
      // x-interface (i1 + 1/2, i2): cells (i2, i1 - G + 1 .. i1 + G)
#pragma unroll
      for (int a = 0; a < 2 * G; ++a)
#pragma unroll
        for (int c = 0; c < NV; ++c) v[c][a] = tile[c][ty + G - 1][tx + a];
      if (st.cfl_mode) {   // the corner's own cell (every cell is the cell of one corner)
        double uc[NV];
#pragma unroll
        for (int c = 0; c < NV; ++c) uc[c] = v[c][G - 1];
        sx = spectral_radius<FLUX, 2, NV>(pb.ph, uc, 0);
        sy = spectral_radius<FLUX, 2, NV>(pb.ph, uc, 1);
      }
      q1 = Select<NV, G, P>::run(v, pb.eps, pb.theta, (pb.flags & FLAG_PSI2_MODIFIED) != 0);
      if (needF) {
        double psi1 = -1.0, al = -1.0;
        if (q1 == 1) {
          psi1 = limiter<NV, G>(v);
          if constexpr (NV == 1) {
            if (pb.flags & FLAG_PSI1_ROE) psi1 = limiter_roe<FLUX, G>(pb.ph, v, 0);
          }
          double uL[NV], uR[NV];
#pragma unroll
          for (int c = 0; c < NV; ++c) {
            uL[c] = v[c][G - 1];
            uR[c] = v[c][G];
          }
          al = fmax(spectral_radius<FLUX, 2, NV>(pb.ph, uL, 0), spectral_radius<FLUX, 2, NV>(pb.ph, uR, 0));
        }
        const int64_t ex = i2 * pb.nIx + (i1 - pb.ioff);
        if (st.recorded) st.ordx[ex] = (int8_t)q1;
        if (st.recorded || q1 == 1) {
          st.psix[ex] = psi1;
          st.alx[ex] = al;
        }
      }
      // y-interface (i1, i2 + 1/2): cells (i2 - G + 1 .. i2 + G, i1)
#pragma unroll
      for (int a = 0; a < 2 * G; ++a)
#pragma unroll
        for (int c = 0; c < NV; ++c) v[c][a] = tile[c][ty + a][tx + G - 1];
      q2 = Select<NV, G, P>::run(v, pb.eps, pb.theta, (pb.flags & FLAG_PSI2_MODIFIED) != 0);
      if (needG) {
        double psi1 = -1.0, al = -1.0;
        if (q2 == 1) {
          psi1 = limiter<NV, G>(v);
          if constexpr (NV == 1) {
            if (pb.flags & FLAG_PSI1_ROE) psi1 = limiter_roe<FLUX, G>(pb.ph, v, 1);
          }
          double uL[NV], uR[NV];
#pragma unroll
          for (int c = 0; c < NV; ++c) {
            uL[c] = v[c][G - 1];
            uR[c] = v[c][G];
          }
          al = fmax(spectral_radius<FLUX, 2, NV>(pb.ph, uL, 1), spectral_radius<FLUX, 2, NV>(pb.ph, uR, 1));
        }
        const int64_t ey = (i2 - pb.ioff) * nx + i1;
        if (st.recorded) st.ordy[ey] = (int8_t)q2;
        if (st.recorded || q2 == 1) {
          st.psiy[ey] = psi1;
          st.aly[ey] = al;
        }
      }
    }
  }
  const int cls = (q1 - 1) * P + (q2 - 1);
  if (inside) st.cls[e] = valid ? (int8_t)cls : (int8_t)-1;
  // square-stencil variant: F in class (q1, q1), G in (q2, q2)
  const bool split = (pb.flags & FLAG_SQUARE_2D) && q1 != q2;
  __shared__ int sh[MAX_CLASSES];
  block_hist(sh, valid, split ? (q1 - 1) * P + (q1 - 1) : cls, st.hist, split ? (q2 - 1) * P + (q2 - 1) : -1);
  if (st.cfl_mode) {
    block_max2(sx, sy);
    if (threadIdx.x == 0) {
      st.part[2 * blockIdx.x] = sx;
      st.part[2 * blockIdx.x + 1] = sy;
    }
  }
}

// f(integral_constant<int, k>) for k = 2, 3, ... in order (the recursion
// levels, each compiled with its own constant k)
template <class F, int... K>
__device__ __forceinline__ void for_levels(F&& f, std::integer_sequence<int, K...>) {
  (f(std::integral_constant<int, K + 2>{}), ...);
}

// One recursion over the rectangle J_Q1 x J_Q2 with time nodes J_QT
// (Taylor order 2 QT).  Each lane is one node (a1, a2) and accumulates the
// series SF = sum_k Fh^{k-1} / k! (DOF) and SG = sum_k Gh^{k-1} / k! (DOG)
// of its node; the fluxes are the eta-weighted sums of SF over row j2 = 0
// and of SG over column j1 = 0.  Same fixed rounding as the 1D kernel.
// g1x, g1y: this node's derivative weights times -lamx and -lamy.
template <int FLUX, int NV, int Q1, int Q2, int QT, bool DOF, bool DOG>
__device__ __forceinline__ void corner_pass(const Phys& ph, const double (&u)[NV],
                                            const double (&f0)[NV], const double (&g0)[NV],
                                            const double* g1x, const double* g1y,
                                            double2* xsb0, double2* xsb1, int stride, int& buf, int slot,
                                            int gbase, int a1, int a2, double (&SF)[NV], double (&SG)[NV]) {
  constexpr int N1 = 2 * Q1;
  constexpr int N2 = 2 * Q2;
  double fc[NV], gc[NV];
#pragma unroll
  for (int c = 0; c < NV; ++c) {
    fc[c] = f0[c];
    gc[c] = g0[c];
    if (DOF) SF[c] = fma(TB.INVFACT[1], f0[c], 0.0);
    if (DOG) SG[c] = fma(TB.INVFACT[1], g0[c], 0.0);
  }
  // Taylor predictions W_r = u + sum_{l<kk} r^l/l! U^l at the time nodes r != 0,
  // extended by one term per level (the same chain of fused multiply-adds as
  // summing from u each level)
  // the row derivative weights of this node in registers for the pass; the
  // column weights too in the order-8 square class (two waves per SIMD with
  // or without them), elsewhere read from LDS at each use (held, they would
  // cost the order-6 square class its third wave per SIMD; the order-4 one
  // ran slower)
  constexpr bool WYR = Q1 == 4 && Q2 == 4;
  double wx[N1], wy[WYR ? N2 : 1];
#pragma unroll
  for (int l = 0; l < N1; ++l) wx[l] = g1x[l];
#pragma unroll
  for (int l = 0; l < (WYR ? N2 : 1); ++l) wy[l] = WYR ? g1y[l] : 0.0;
  double W[2 * QT][NV];
#pragma unroll
  for (int ri = 0; ri < 2 * QT; ++ri)
#pragma unroll
    for (int c = 0; c < NV; ++c) W[ri][c] = u[c];
  // one recursion level: exchange Fh^{kk-2}, Gh^{kk-2}; U^{kk-1}; predictions;
  // Fh^{kk-1}, Gh^{kk-1} and their series terms (each level compiled with
  // its own constant kk)
  auto level = [&](auto kkc) {
    constexpr int kk = decltype(kkc)::value;
    double2* xsw = buf ? xsb1 : xsb0;
    Xch<NV>::put(xsw, stride, slot, fc, gc);
    Groups<(2 * Q1) * (2 * Q2)>::sync();
    buf ^= 1;
    const double* xr = reinterpret_cast<const double*>(xsw);
    // U^{kk-1} = -lamx d_x Fh^{kk-2} - lamy d_y Gh^{kk-2} at this node: one
    // chain of fused multiply-adds over the row (x) and then the column (y)
    double Uk[NV];
#pragma unroll
    for (int c = 0; c < NV; ++c) {
      double s = 0.0;
#pragma unroll
      for (int l = 0; l < N1; ++l) s = fma(wx[l], Xch<NV>::get(xr, stride, gbase + a2 * N1 + l, c, false), s);
#pragma unroll
      for (int l = 0; l < N2; ++l)
        s = fma(WYR ? wy[WYR ? l : 0] : g1y[l], Xch<NV>::get(xr, stride, gbase + l * N1 + a1, c, true), s);
      Uk[c] = s;
    }
#pragma unroll
    for (int ri = 0; ri < 2 * QT; ++ri) {
      const int r = ri - QT + 1;
      if (r == 0) continue;
#pragma unroll
      for (int c = 0; c < NV; ++c) W[ri][c] = fma(TB.TAYLOR[r + PMAX - 1][kk - 1], Uk[c], W[ri][c]);
    }
    double nf[NV], ng[NV];
#pragma unroll
    for (int c = 0; c < NV; ++c) {
      nf[c] = 0.0;
      ng[c] = 0.0;
    }
    // Euler: the reciprocal densities of all predicted states first, their
    // Newton steps interleaved (time node r = 0 is the node state: its flux
    // is f0, g0)
    double rho[2 * QT - 1], ir[2 * QT - 1];
    if constexpr (FLUX == EUL) {
#pragma unroll
      for (int ri = 0; ri < 2 * QT; ++ri)
        if (ri != QT - 1) rho[ri < QT - 1 ? ri : ri - 1] = W[ri][0];
      recip_n(rho, ir);
    }
#pragma unroll
    for (int ri = 0; ri < 2 * QT; ++ri) {
      const int r = ri - QT + 1;
      // a time node whose weight is exactly zero adds nothing to Fh, Gh: its
      // fluxes (and reciprocal density) are not evaluated (the same sums
      // for finite values)
      if (TB.GT[QT][kk - 1][ri] == 0.0) continue;
      double pf[NV], pg[NV];
      if (r == 0) {
#pragma unroll
        for (int c = 0; c < NV; ++c) {
          pf[c] = f0[c];
          pg[c] = g0[c];
        }
      } else if constexpr (FLUX == EUL) {
        euler2d_ir(ph, W[ri], ir[ri < QT - 1 ? ri : ri - 1], pf, pg);
      } else {
        flux2d<FLUX, NV>(ph, W[ri], pf, pg);
      }
#pragma unroll
      for (int c = 0; c < NV; ++c) {
        nf[c] = fma(TB.GT[QT][kk - 1][ri], pf[c], nf[c]);
        ng[c] = fma(TB.GT[QT][kk - 1][ri], pg[c], ng[c]);
      }
    }
#pragma unroll
    for (int c = 0; c < NV; ++c) {
      fc[c] = nf[c];
      gc[c] = ng[c];
      if (DOF) SF[c] = fma(TB.INVFACT[kk], nf[c], SF[c]);
      if (DOG) SG[c] = fma(TB.INVFACT[kk], ng[c], SG[c]);
    }
  };
  for_levels(level, std::make_integer_sequence<int, 2 * QT - 1>{});
}

// Exchange slots of a group of L = (2 q1)(2 q2) corner nodes: node (a1, a2)
// of group g at g GS + a2 (2 q1) + a1.  Groups of 36 nodes (class (3, 3))
// start 38 slots apart: 36 apart, the first rows of two groups that share a
// 16-lane phase of a 128-bit LDS access fall on the same banks.
template <int L>
constexpr int corner_group_stride() {
  return L == 36 ? L + 2 : L;
}

// slots per exchange plane (spare groups of idle lanes included)
template <int L>
constexpr int corner_stride() {
  return Groups<L>::TOTAL * corner_group_stride<L>();
}

// Fluxes of the corners of order class (Q1, Q2) (Sec. 4; rectangle J_Q1 x J_Q2),
// items [base, end) of the list; every class but (1,1), which runs one lane
// per corner (flux2d_q11).  SQUARE: list entries carry the square-stencil
// variant's tags (square classes only).  xsm: the two exchange buffers
// (2 Xch<NV>::NP corner_stride<L>() double2), gxs, gys: the derivative weights
// (EdgeWeights), in LDS.
template <int FLUX, int NV, int Q1, int Q2, bool SQUARE>
__device__ __forceinline__ void flux2d_body(const KProb& pb, const KStep& st, int tid, double dt,
                                            const int32_t* items, int base, int end, double2* xsm, const double* gxs,
                                            const double* gys) {
  static_assert(Q1 > 1 || Q2 > 1, "class (1,1) runs in flux2d_q11");
  constexpr int N1 = 2 * Q1, N2 = 2 * Q2, L = N1 * N2;
  using Grp = Groups<L>;
  constexpr int NP = Xch<NV>::NP;
  constexpr int STRIDE = corner_stride<L>();
  constexpr int GS = corner_group_stride<L>();
  double2* const xs[2] = {xsm, xsm + NP * STRIDE};

  const Grp grp(tid);
  const int g = grp.g;
  const int nd = grp.node;
  const int a1 = nd % N1, a2 = nd / N1;     // node (j1, j2) = (a1 - Q1 + 1, a2 - Q2 + 1)
  const bool inblk = grp.in;
  const int64_t nx = pb.nx, ny = pb.ny, plane = pb.nx * pb.ny;
  const int nx32 = (int)pb.nx, ny32 = (int)pb.ny, ioff = (int)pb.ioff;
  const uint32_t n1u = (uint32_t)pb.n1;
  // the corner pass holds a node's row weights in registers and reads its
  // column weights at each use
  const double* g1x = gxs + EdgeWeights::first(Q1) + a1 * N1;
  const double* g1y = gys + EdgeWeights::first(Q2) + a2 * N2;

  int buf = 0;
  for (; base < end; base += Grp::PER_BLOCK) {
    {
      const bool valid = inblk && base + g < end;
      const int32_t raw = valid ? items[base + g] : 0;
      // square-stencil variant: entries carry which flux to store (1 F, 2 G, 0 both)
      const int32_t e = SQUARE ? (raw & ((1 << LIST_TAG_SHIFT) - 1)) : raw;
      const int tag = SQUARE ? (raw >> LIST_TAG_SHIFT) : 0;
      const uint32_t eq = (uint32_t)e / n1u;
      const int i2 = (int)eq + ioff, i1 = (int)((uint32_t)e - eq * n1u) + ioff;
      const int x = bc_index32(i1 + (a1 - Q1 + 1), nx32, pb.bc);
      const int y = bc_index32(i2 + (a2 - Q2 + 1), ny32, pb.bc);
      const double* un = st.u + ((int64_t)y * nx + x);
      double u[NV];
#pragma unroll
      for (int c = 0; c < NV; ++c) u[c] = valid ? un[c * plane] : 1.0;
      double f0[NV], g0[NV];
      flux2d<FLUX, NV>(pb.ph, u, f0, g0);
      double SF[NV], SG[NV];
      const int slot = g * GS + nd;
      if constexpr (Q1 == Q2) {
        corner_pass<FLUX, NV, Q1, Q2, Q1, true, true>(pb.ph, u, f0, g0, g1x, g1y, xs[0], xs[1],
                                                      STRIDE, buf, slot, g * GS, a1, a2, SF, SG);
      } else {
        corner_pass<FLUX, NV, Q1, Q2, Q1, true, false>(pb.ph, u, f0, g0, g1x, g1y, xs[0], xs[1],
                                                       STRIDE, buf, slot, g * GS, a1, a2, SF, SG);
        corner_pass<FLUX, NV, Q1, Q2, Q2, false, true>(pb.ph, u, f0, g0, g1x, g1y, xs[0], xs[1],
                                                       STRIDE, buf, slot, g * GS, a1, a2, SF, SG);
      }
      // F_c = sum_l eta_l SF_(l,0),c and G_c = sum_l eta_l SG_(0,l),c on 2 NV lanes
      {
        double2* xsw = buf ? xs[1] : xs[0];
        Xch<NV>::put(xsw, STRIDE, slot, SF, SG);
        Grp::sync();
      }
      const double* xr = reinterpret_cast<const double*>(buf ? xs[1] : xs[0]);
      double acc[2] = {0.0, 0.0};
#pragma unroll
      for (int tk = 0; tk < 2; ++tk) {
        const int task = nd + tk * L;
        if (!valid || task >= 2 * NV) continue;
        const bool isG = task >= NV;
        const int c = isG ? task - NV : task;
        double t = 0.0;
        if (!isG) {
#pragma unroll
          for (int l = 0; l < N1; ++l) t = fma(TB.ETA[Q1][l], Xch<NV>::get(xr, STRIDE, g * GS + (Q2 - 1) * N1 + l, c, false), t);
        } else {
#pragma unroll
          for (int l = 0; l < N2; ++l) t = fma(TB.ETA[Q2][l], Xch<NV>::get(xr, STRIDE, g * GS + l * N1 + (Q1 - 1), c, true), t);
        }
        acc[tk] = t;
      }
      buf ^= 1;   // the assembly may still read this buffer
      // finish and store the assembled components
#pragma unroll
      for (int tk = 0; tk < 2; ++tk) {
        const int task = nd + tk * L;
        if (!valid || task >= 2 * NV) continue;
        const bool isG = task >= NV;
        const int c = isG ? task - NV : task;
        // transmissive ghost corners need one flux only; tagged entries one flux each
        const bool need = isG ? (i1 >= 0 && tag != 1) : (i2 >= 0 && tag != 2);
        if (!need) continue;
        double v = acc[tk];
        if ((!isG && Q1 == 1) || (isG && Q2 == 1)) {
          // 2D FL-CAT2 (Sec. 4): psi^1 CAT2 + (1 - psi^1) Rusanov in this direction
          const int64_t x0 = bc_index32(i1, nx32, pb.bc), y0 = bc_index32(i2, ny32, pb.bc);
          const int64_t xr = isG ? x0 : bc_index32(i1 + 1, nx32, pb.bc);
          const int64_t yr = isG ? bc_index32(i2 + 1, ny32, pb.bc) : y0;
          const int64_t ei = isG ? (int64_t)(i2 - ioff) * nx + i1 : (int64_t)i2 * pb.nIx + (i1 - ioff);
          const double psi = isG ? st.psiy[ei] : st.psix[ei];
          const double al = isG ? st.aly[ei] : st.alx[ei];
          double uL[NV], uR[NV], fL[NV], gL[NV], fR[NV], gR[NV];
#pragma unroll
          for (int cc = 0; cc < NV; ++cc) {
            uL[cc] = st.u[(cc * ny + y0) * nx + x0];
            uR[cc] = st.u[(cc * ny + yr) * nx + xr];
          }
          flux2d<FLUX, NV>(pb.ph, uL, fL, gL);
          flux2d<FLUX, NV>(pb.ph, uR, fR, gR);
          double ul = 0.0, ur = 0.0, hl = 0.0, hr = 0.0;
#pragma unroll
          for (int cc = 0; cc < NV; ++cc)
            if (cc == c) {
              ul = uL[cc];
              ur = uR[cc];
              hl = isG ? gL[cc] : fL[cc];
              hr = isG ? gR[cc] : fR[cc];
            }
          const double alf = (isG ? pb.dy : pb.dx) / ((double)pb.dim * dt);
          const double lo = lo_flux<FLUX, 2, NV>(pb.ph, pb.flags, isG ? 1 : 0, uL, uR, hl, hr, ul, ur, al, alf);
          v = psi * v + (1.0 - psi) * lo;
        }
        if (isG) st.Gy[((int64_t)c * pb.nIy + (i2 - ioff)) * nx + i1] = v;
        else st.Fx[((int64_t)c * ny + i2) * pb.nIx + (i1 - ioff)] = v;
      }
    }
  }
}


// Order class (1,1) with ONE LANE PER CORNER.  The corner's four nodes
// (j1, j2) in {0,1}^2 (cells (i1 + j1, i2 + j2)) live in one lane, which
// computes, with the same operations in the same order as the node-per-lane
// kernel, just the quantities the corner's fluxes read (Sec. 4 with
// q1 = q2 = 1: one recursion level): the point fluxes at the four nodes, U^1
// at the three nodes of row j2 = 0 and column j1 = 0, the flux at their
// Taylor predictions, the series of F on the row and of G on the column,
// the eta-weighted sums and the FL-CAT2 blends.  No LDS exchange and no
// barrier; a wavefront holds 64 independent corners.
template <int FLUX, int NV, bool SQUARE>
__device__ __forceinline__ void flux2d_q11(const KProb& pb, const KStep& st, int tid, double dt, const int32_t* items,
                                           int base, int end) {
  const double lamx = dt / pb.dx, lamy = dt / pb.dy;
  // derivative weights times -lamx (x) and -lamy (y): gx[a][l], gy[a][l]
  double gx[2][2], gy[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int l = 0; l < 2; ++l) {
      gx[a][l] = -lamx * TB.G1[1][a][l];
      gy[a][l] = -lamy * TB.G1[1][a][l];
    }
  const double tay = TB.TAYLOR[PMAX][1];                      // r = 1, first term
  const double gt0 = TB.GT[1][1][0], gt1 = TB.GT[1][1][1];    // time derivative weights at r = 0, 1
  const int64_t nx = pb.nx, ny = pb.ny, plane = pb.nx * pb.ny;
  const int nx32 = (int)pb.nx, ny32 = (int)pb.ny, ioff = (int)pb.ioff;
  const uint32_t n1u = (uint32_t)pb.n1;
  for (int it = base + tid; it < end; it += BLOCK) {
    const int32_t raw = items[it];
    const int32_t e = SQUARE ? (raw & ((1 << LIST_TAG_SHIFT) - 1)) : raw;
    const int tag = SQUARE ? (raw >> LIST_TAG_SHIFT) : 0;
    const uint32_t eq = (uint32_t)e / n1u;
    const int i2 = (int)eq + ioff, i1 = (int)((uint32_t)e - eq * n1u) + ioff;
    int xs[2], ys[2];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      xs[a] = bc_index32(i1 + a, nx32, pb.bc);
      ys[a] = bc_index32(i2 + a, ny32, pb.bc);
    }
    // node states and point fluxes, [j2][j1]
    double u[2][2][NV], f0[2][2][NV], g0[2][2][NV];
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int a = 0; a < 2; ++a) {
#pragma unroll
        for (int c = 0; c < NV; ++c) u[b][a][c] = st.u[c * plane + (int64_t)ys[b] * nx + xs[a]];
        flux2d<FLUX, NV>(pb.ph, u[b][a], f0[b][a], g0[b][a]);
      }
    // series of F on the row j2 = 0 (nodes (0,0), (1,0)) and of G on the
    // column j1 = 0 (nodes (0,0), (0,1)): S = Fh^0 / 1! + Fh^1 / 2!
    double SF[2][NV], SG[2][NV];
#pragma unroll
    for (int n = 0; n < 3; ++n) {
      const int a = n == 1 ? 1 : 0, b = n == 2 ? 1 : 0;   // nodes (0,0), (1,0), (0,1)
      double w[NV];
#pragma unroll
      for (int c = 0; c < NV; ++c) {
        // U^1 = -lamx d_x Fh^0 - lamy d_y Gh^0: one chain, row then column
        double s = 0.0;
        s = fma(gx[a][0], f0[b][0][c], s);
        s = fma(gx[a][1], f0[b][1][c], s);
        s = fma(gy[b][0], g0[0][a][c], s);
        s = fma(gy[b][1], g0[1][a][c], s);
        w[c] = fma(tay, s, u[b][a][c]);
      }
      double pf[NV], pg[NV];
      flux2d<FLUX, NV>(pb.ph, w, pf, pg);
#pragma unroll
      for (int c = 0; c < NV; ++c) {
        if (b == 0) {   // on the row: F's series
          const double nf = fma(gt1, pf[c], fma(gt0, f0[b][a][c], 0.0));
          SF[a][c] = fma(TB.INVFACT[2], nf, fma(TB.INVFACT[1], f0[b][a][c], 0.0));
        }
        if (a == 0) {   // on the column: G's series
          const double ng = fma(gt1, pg[c], fma(gt0, g0[b][a][c], 0.0));
          SG[b][c] = fma(TB.INVFACT[2], ng, fma(TB.INVFACT[1], g0[b][a][c], 0.0));
        }
      }
    }
    const bool needF = i2 >= 0 && tag != 2, needG = i1 >= 0 && tag != 1;
    if (needF) {
      // F: eta-weighted row sum, FL-CAT2 blend with the nodes (0,0), (1,0)
      const int64_t ei = (int64_t)i2 * pb.nIx + (i1 - ioff);
      const double psi = st.psix[ei], al = st.alx[ei];
      const double alf = pb.dx / ((double)pb.dim * dt);
#pragma unroll
      for (int c = 0; c < NV; ++c) {
        double v = fma(TB.ETA[1][1], SF[1][c], fma(TB.ETA[1][0], SF[0][c], 0.0));
        const double lo = lo_flux<FLUX, 2, NV>(pb.ph, pb.flags, 0, u[0][0], u[0][1], f0[0][0][c], f0[0][1][c],
                                               u[0][0][c], u[0][1][c], al, alf);
        v = psi * v + (1.0 - psi) * lo;
        st.Fx[((int64_t)c * ny + i2) * pb.nIx + (i1 - ioff)] = v;
      }
    }
    if (needG) {
      const int64_t ei = (int64_t)(i2 - ioff) * nx + i1;
      const double psi = st.psiy[ei], al = st.aly[ei];
      const double alf = pb.dy / ((double)pb.dim * dt);
#pragma unroll
      for (int c = 0; c < NV; ++c) {
        double v = fma(TB.ETA[1][1], SG[1][c], fma(TB.ETA[1][0], SG[0][c], 0.0));
        const double lo = lo_flux<FLUX, 2, NV>(pb.ph, pb.flags, 1, u[0][0], u[1][0], g0[0][0][c], g0[1][0][c],
                                               u[0][0][c], u[1][0][c], al, alf);
        v = psi * v + (1.0 - psi) * lo;
        st.Gy[((int64_t)c * pb.nIy + (i2 - ioff)) * nx + i1] = v;
      }
    }
  }
}

// The order classes of a 2D step in one or two launches, by the blocks that
// fit a CU at their register need: three (THREE: orders up to 3 but (2, 3)
// and (3, 2); up to 168 registers per lane), two (TWO: those two and the
// classes with an order 4; up to 256), or all of them at two (ALL).  All the
// classes of a launch share its blocks
// (Chunks), so that a small grid's classes run side by side and a large one's
// leave no tails.  The costliest class comes first.  Against one launch per
// class or mirror pair, a step of 64^2 corners at P = 3 34.3 -> 27.7 us, 192^2
// 74.6 -> 59.0, 400^2 at P = 2 79.7 -> 71.7, 1000^2 at P = 3 1213 -> 1180, 2048^2
// 6401 -> 6407 (the gain of the tails is spent on registers: 12 spilled of the
// 168 that three blocks per CU allow), 1021 x 777 at P = 4 3222 -> 3169.
struct Cls {
  int q1, q2;
};
enum Blocks { THREE, TWO, ALL };
template <int P, Blocks B, bool SQUARE>
struct ClassSet {
  static constexpr Cls EVERY[MAX_CLASSES] = {{4, 4}, {3, 4}, {4, 3}, {2, 4}, {4, 2}, {1, 4}, {4, 1}, {2, 3},
                                             {3, 2}, {3, 3}, {1, 3}, {3, 1}, {2, 2}, {1, 2}, {2, 1}, {1, 1}};
  static constexpr bool few(Cls c) { return c.q1 == 4 || c.q2 == 4 || c.q1 + c.q2 == 5; }
  static constexpr bool has(Cls c) {
    return c.q1 <= P && c.q2 <= P && (B == ALL || few(c) == (B == TWO)) && (!SQUARE || c.q1 == c.q2);
  }
  static constexpr int count() {
    int n = 0;
    for (Cls c : EVERY) n += has(c);
    return n;
  }
  static constexpr int N = count();
  static constexpr Cls at(int k) {
    for (Cls c : EVERY)
      if (has(c) && k-- == 0) return c;
    return {1, 1};
  }
  static constexpr int per_round(Cls c) {
    switch (4 * c.q1 * c.q2) {
      case 4: return BLOCK;
      case 8: return Groups<8>::PER_BLOCK;
      case 12: return Groups<12>::PER_BLOCK;
      case 16: return Groups<16>::PER_BLOCK;
      case 24: return Groups<24>::PER_BLOCK;
      case 32: return Groups<32>::PER_BLOCK;
      case 36: return Groups<36>::PER_BLOCK;
      case 48: return Groups<48>::PER_BLOCK;
      default: return Groups<64>::PER_BLOCK;
    }
  }
  static constexpr int stride(Cls c) {
    switch (4 * c.q1 * c.q2) {
      case 4: return 0;
      case 8: return corner_stride<8>();
      case 12: return corner_stride<12>();
      case 16: return corner_stride<16>();
      case 24: return corner_stride<24>();
      case 32: return corner_stride<32>();
      case 36: return corner_stride<36>();
      case 48: return corner_stride<48>();
      default: return corner_stride<64>();
    }
  }
  static constexpr int max_stride() {
    int m = 1;
    for (int k = 0; k < N; ++k) m = stride(at(k)) > m ? stride(at(k)) : m;
    return m;
  }
  static constexpr int min_per_round() {
    int m = BLOCK;
    for (int k = 0; k < N; ++k) m = per_round(at(k)) < m ? per_round(at(k)) : m;
    return m;
  }
};

// waves per SIMD the kernel is held to: a scalar law's P = 2 six (99 registers
// otherwise, four; 800^2 to 2000^2 4 to 5 % faster)
template <int NV, int P, Blocks B>
constexpr int flux2d_waves() {
  return NV == 1 && P == 2 ? 6 : B == THREE ? 3 : 2;
}

template <int FLUX, int NV, int P, Blocks B, bool SQUARE, bool DRAW>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(flux2d_waves<NV, P, B>()))) void k_flux2d(
    KProb pb, KStep st) {
  using Set = ClassSet<P, B, SQUARE>;
  static_assert(Set::N <= 9, "one case of the switch per class");
  __shared__ double2 xsm[2 * Xch<NV>::NP * Set::max_stride()];
  __shared__ double gxs[EdgeWeights::first(P + 1)], gys[EdgeWeights::first(P + 1)];
  __shared__ ChunkTable tab;
  const double dt = step_dt(st);
  for (int q = 1; q <= P; ++q) {
    const double lamx = dt / pb.dx, lamy = dt / pb.dy;
    for (int i = threadIdx.x; i < 4 * q * q; i += BLOCK) {
      const double w = TB.G1[q][i / (2 * q)][i % (2 * q)];
      gxs[EdgeWeights::first(q) + i] = -lamx * w;
      gys[EdgeWeights::first(q) + i] = -lamy * w;
    }
  }
  constexpr auto sets = [] {
    struct {
      int cls[MAX_CLASSES], per_round[MAX_CLASSES];
    } t{};
    for (int k = 0; k < Set::N; ++k) {
      t.cls[k] = (Set::at(k).q1 - 1) * P + Set::at(k).q2 - 1;
      t.per_round[k] = Set::per_round(Set::at(k));
    }
    return t;
  }();
  constexpr int MIN = NV == 1 && P == 2 ? 2 : 1;
  Chunks<Set::N, DRAW, MIN> ck(st, tab, B == TWO ? 1 : 0, blockIdx.x, gridDim.x, [&](int k, int& c, int& per_round) {
    c = sets.cls[k];
    per_round = sets.per_round[k];
  });
  auto run = [&](auto kc) {
    constexpr int k = decltype(kc)::value;
    if constexpr (k < Set::N) {
      constexpr Cls c = Set::at(k);
      // what a class derives from its lane's number and the time step is
      // computed at each chunk: kept for all classes at once it would spill
      int tid = threadIdx.x;
      double h = dt;
      asm volatile("" : "+v"(tid), "+v"(h));
      if constexpr (c.q1 == 1 && c.q2 == 1)
        flux2d_q11<FLUX, NV, SQUARE>(pb, st, tid, h, ck.items, ck.base, ck.end);
      else
        flux2d_body<FLUX, NV, c.q1, c.q2, SQUARE>(pb, st, tid, h, ck.items, ck.base, ck.end, xsm, gxs, gys);
    }
  };
  while (ck.start(st, tab)) {
    switch (ck.cls) {
      case 0: run(std::integral_constant<int, 0>{}); break;
      case 1: run(std::integral_constant<int, 1>{}); break;
      case 2: run(std::integral_constant<int, 2>{}); break;
      case 3: run(std::integral_constant<int, 3>{}); break;
      case 4: run(std::integral_constant<int, 4>{}); break;
      case 5: run(std::integral_constant<int, 5>{}); break;
      case 6: run(std::integral_constant<int, 6>{}); break;
      case 7: run(std::integral_constant<int, 7>{}); break;
      default: run(std::integral_constant<int, 8>{}); break;
    }
    ck.advance(tab);
  }
}

template <int FLUX, int NV>
__global__ __launch_bounds__(BLOCK) void k_update2d(KProb pb, KStep st) {
  const int64_t e = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  const int64_t nx = pb.nx, ny = pb.ny;
  if (e >= nx * ny) return;
  const int64_t i1 = e % nx, i2 = e / nx;
  const double dt = step_dt(st);
  const double lamx = dt / pb.dx, lamy = dt / pb.dy;
  const int64_t kxr = i1 - pb.ioff, kxl = (pb.bc == PERIODIC) ? (i1 == 0 ? nx - 1 : i1 - 1) : i1;
  const int64_t kyr = i2 - pb.ioff, kyl = (pb.bc == PERIODIC) ? (i2 == 0 ? ny - 1 : i2 - 1) : i2;
  double w[NV];
  bool finite = true;
#pragma unroll
  for (int c = 0; c < NV; ++c) {
    const double Fl = st.Fx[(c * ny + i2) * pb.nIx + kxl], Fr = st.Fx[(c * ny + i2) * pb.nIx + kxr];
    const double Gl = st.Gy[(c * pb.nIy + kyl) * nx + i1], Gr = st.Gy[(c * pb.nIy + kyr) * nx + i1];
    const int64_t idx = (c * ny + i2) * nx + i1;
    w[c] = st.u[idx] + lamx * (Fl - Fr) + lamy * (Gl - Gr);
    st.uout[idx] = w[c];
    finite = finite && isfinite(w[c]);
  }
  uint32_t bad = (finite ? 0u : 1u) | (physical<FLUX, 2, NV>(pb.ph, w) ? 0u : 2u);
  if (bad) atomicOr(st.status, bad);
}

// ====================================================================== CFL
template <int FLUX, int DIM, int NV>
__global__ __launch_bounds__(BLOCK) void k_max_speed(KProb pb, const double* __restrict__ u,
                                                     unsigned long long* smax) {
  const int64_t n = pb.nx * (DIM == 2 ? pb.ny : 1);
  double m0 = 0.0, m1 = 0.0;
  for (int64_t e = (int64_t)blockIdx.x * BLOCK + threadIdx.x; e < n; e += (int64_t)gridDim.x * BLOCK) {
    double w[NV];
#pragma unroll
    for (int c = 0; c < NV; ++c) w[c] = u[c * n + e];
    m0 = fmax(m0, spectral_radius<FLUX, DIM, NV>(pb.ph, w, 0));
    if (DIM == 2) m1 = fmax(m1, spectral_radius<FLUX, DIM, NV>(pb.ph, w, 1));
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    m0 = fmax(m0, __shfl_xor(m0, off));
    m1 = fmax(m1, __shfl_xor(m1, off));
  }
  __shared__ double red[2][BLOCK / 64];
  if (__lane_id() == 0) {
    red[0][threadIdx.x >> 6] = m0;
    red[1][threadIdx.x >> 6] = m1;
  }
  __syncthreads();
  // one atomic per block; the bit patterns of non-negative doubles order like the values
  if (threadIdx.x == 0) {
#pragma unroll
    for (int w = 1; w < BLOCK / 64; ++w) {
      m0 = fmax(m0, red[0][w]);
      m1 = fmax(m1, red[1][w]);
    }
    atomicMax(&smax[0], (unsigned long long)__double_as_longlong(m0));
    if (DIM == 2) atomicMax(&smax[1], (unsigned long long)__double_as_longlong(m1));
  }
}

__global__ void k_cfl_dt(int dim, double dx, double dy, const double* smax, double cfl, double t_final,
                         double* t_dev, double* dt_dev) {
  cfl_rule(dim, dx, dy, smax[0], dim == 2 ? smax[1] : 0.0, cfl, t_final, t_dev, dt_dev);
}


// ================================================================ launchers
CflReduce cfl_reduce(const KProb& pb, const KStep& st, int nparts) {
  CflReduce r{};
  if (st.cfl_mode) {
    r.part = st.part;
    r.nparts = nparts;
    r.dim = pb.dim;
    r.dx = pb.dx;
    r.dy = pb.dy;
    r.cfl = st.cfl;
    r.t_final = st.t_final;
    r.t_dev = st.t_dev;
    r.dt_out = st.dt_out;
  }
  return r;
}

#define ACAT_CHECK_LAUNCH()                  \
  do {                                       \
    hipError_t e_ = hipGetLastError();       \
    if (e_ != hipSuccess) return e_;         \
  } while (0)

// The classes of one launch (ClassSet).
template <int FLUX, int NV, int P, Blocks B, bool SQUARE, bool DRAW = true>
hipError_t launch_flux2d(const KProb& pb, const KStep& st, int cap, hipStream_t s) {
  using Set = ClassSet<P, B, SQUARE>;
  if constexpr (Set::N > 0) {
    static constexpr LaunchName name = class_launch_name<Set>("flux2d_");
    auto kern = k_flux2d<FLUX, NV, P, B, SQUARE, DRAW>;
    static const int per_cu = [&] {
      int b = 0;
      return hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, kern, BLOCK, 0) == hipSuccess && b > 0 ? b : 1;
    }();
    // no more blocks than rounds, with one cut short per class and XCD
    const int64_t rounds = pb.n1 * pb.n2 / Set::min_per_round() + NXCD * Set::N;
    const int grid = persistent_grid(kern, rounds * BLOCK, cap, BLOCK, per_cu);
    {
      ProfScope ps(name.s, s);
      kern<<<grid, BLOCK, 0, s>>>(pb, st);
    }
    ACAT_CHECK_LAUNCH();
  }
  return hipSuccess;
}

// Up to P = 2 every class fits three blocks per CU.  Above, those that do not
// are a launch of their own, but on grids so small that the launch costs more
// than the third block gives: at P = 3 a step of 64^2 corners takes 25.2 us in
// one launch and 28.0 in two, 192^2 51.5 and 59.7, 256^2 90.7 and 97.9, 320^2
// 149 and 149, 512^2 358 and 343.  (At P = 4 two are as fast or faster: 100^2
// 37.2 and 34.9, 300^2 193.8 and 195.6, 1021 x 777 3391 and 3397.)
constexpr int64_t ONE_LAUNCH = 90000;
// A scalar law's rounds of P <= 2 take about as long as a ticket: drawn one by one
// they made advection 500^2 P = 2 67 us without noise, where a launch per class took
// 61, and 1200^2 P = 1 64 (63).  P = 1 takes fixed shares (55; one class, whose rounds
// are alike), P = 2 up to this many corners: 300^2 fixed / tickets of two rounds and
// more 29 / 34 us, 400^2 41 / 44, 500^2 58 / 57, 600^2 78 / 75, 900^2 155 / 133.
constexpr int64_t SCALAR_FIXED = 250000;
template <int FLUX, int NV, int P, bool SQUARE>
hipError_t launch_classes2d(const KProb& pb, const KStep& st, int cap, hipStream_t s) {
  if constexpr (NV == 1 && P == 1) {
    return launch_flux2d<FLUX, NV, P, THREE, SQUARE, false>(pb, st, cap, s);
  } else {
    if constexpr (NV == 1 && P == 2) {
      if (pb.n1 * pb.n2 <= SCALAR_FIXED) return launch_flux2d<FLUX, NV, P, THREE, SQUARE, false>(pb, st, cap, s);
    }
    if constexpr (P == 3) {
      if (pb.n1 * pb.n2 <= ONE_LAUNCH) return launch_flux2d<FLUX, NV, P, ALL, SQUARE>(pb, st, cap, s);
    }
    const hipError_t e = launch_flux2d<FLUX, NV, P, THREE, SQUARE>(pb, st, cap, s);
    return e != hipSuccess ? e : launch_flux2d<FLUX, NV, P, TWO, SQUARE>(pb, st, cap, s);
  }
}

// Tiles up to which the list kernel sums the class histograms itself instead of
// reading the prefix that one launch more makes.  Each block then reads the
// histograms of all tiles (from L2), work that grows with the tiles' square.  Whole
// step, Euler, two launches / one: 64^2 P = 3 25.3 us / 24.3, 128^2 P = 2 23.8 / 21.4,
// 400^2 P = 2 (625 tiles) 70.5 / 68.4, P = 4 578 / 578, 512^2 P = 1 40.5 / 38.7; beyond
// the line 640^2 P = 2 (1600) 146.5 / 145.3.  The loads go eight at a time: one by
// one 800^2 took 222 us, against 209 in two launches.
constexpr int LISTS_ONE_LAUNCH = 1024;

template <int FLUX, int NV, int P>
hipError_t lists2d_impl(const KProb& pb, const KStep& st, hipStream_t s) {
  const int cblocks = (int)class_tiles(pb);
  {
    ProfScope ps("classify2d", s);
    k_classify2d<FLUX, NV, P><<<cblocks, BLOCK, 0, s>>>(pb, st);
  }
  ACAT_CHECK_LAUNCH();
  {
    ProfScope ps("class_lists", s);
    const bool square = (pb.flags & FLAG_SQUARE_2D) != 0;
    const CflReduce cr = cfl_reduce(pb, st, cblocks);
    if (cblocks <= LISTS_ONE_LAUNCH) {
      auto kern = square ? k_scatter<P * P, true, true, true> : k_scatter<P * P, true, false, true>;
      kern<<<cblocks + (st.cfl_mode ? 1 : 0), BLOCK, 0, s>>>(st.cls, 0, pb.n1, pb.n2, cblocks, st.offs, st.counts,
                                                             st.list, P, st.hist, st.tickets, cr);
    } else {
      k_scan_hist<<<P * P + (st.cfl_mode ? 1 : 0), SCAN_T, 0, s>>>(st.hist, cblocks, st.offs, st.counts, P * P, cr,
                                                                  st.tickets);
      auto kern = square ? k_scatter<P * P, true, true> : k_scatter<P * P, true>;
      kern<<<cblocks, BLOCK, 0, s>>>(st.cls, 0, pb.n1, pb.n2, cblocks, st.offs, st.counts, st.list, P, nullptr,
                                     nullptr, {});
    }
  }
  ACAT_CHECK_LAUNCH();
  return hipSuccess;
}

template <int FLUX, int NV, int P>
hipError_t step2d_impl(const KProb& pb, const KStep& st, int cap, hipStream_t s) {
  hipError_t e;
  if ((e = lists2d_impl<FLUX, NV, P>(pb, st, s)) != hipSuccess) return e;
  e = pb.flags & FLAG_SQUARE_2D ? launch_classes2d<FLUX, NV, P, true>(pb, st, cap, s)
                                : launch_classes2d<FLUX, NV, P, false>(pb, st, cap, s);
  if (e != hipSuccess) return e;
  {
    ProfScope ps("update2d", s);
    k_update2d<FLUX, NV><<<(unsigned)((pb.nx * pb.ny + BLOCK - 1) / BLOCK), BLOCK, 0, s>>>(pb, st);
  }
  ACAT_CHECK_LAUNCH();
  return hipSuccess;
}

}  // namespace

hipError_t launch_step_2d(const KProb& pb, const KStep& st, int grid_blocks, hipStream_t s) {
  const int cap = grid_blocks;
  if (pb.flux == EUL) {
    switch (pb.P) {
      case 1: return step2d_impl<EUL, 4, 1>(pb, st, cap, s);
      case 2: return step2d_impl<EUL, 4, 2>(pb, st, cap, s);
      case 3: return step2d_impl<EUL, 4, 3>(pb, st, cap, s);
      case 4: return step2d_impl<EUL, 4, 4>(pb, st, cap, s);
    }
  } else if (pb.flux == ADV) {
    switch (pb.P) {
      case 1: return step2d_impl<ADV, 1, 1>(pb, st, cap, s);
      case 2: return step2d_impl<ADV, 1, 2>(pb, st, cap, s);
      case 3: return step2d_impl<ADV, 1, 3>(pb, st, cap, s);
      case 4: return step2d_impl<ADV, 1, 4>(pb, st, cap, s);
    }
  }
  return hipErrorInvalidValue;
}

hipError_t launch_lists(const KProb& pb, const KStep& st, hipStream_t s) {
  if (pb.flux == EUL) {
    switch (pb.P) {
      case 1: return lists2d_impl<EUL, 4, 1>(pb, st, s);
      case 2: return lists2d_impl<EUL, 4, 2>(pb, st, s);
      case 3: return lists2d_impl<EUL, 4, 3>(pb, st, s);
      case 4: return lists2d_impl<EUL, 4, 4>(pb, st, s);
    }
  } else if (pb.flux == ADV) {
    switch (pb.P) {
      case 1: return lists2d_impl<ADV, 1, 1>(pb, st, s);
      case 2: return lists2d_impl<ADV, 1, 2>(pb, st, s);
      case 3: return lists2d_impl<ADV, 1, 3>(pb, st, s);
      case 4: return lists2d_impl<ADV, 1, 4>(pb, st, s);
    }
  }
  return hipErrorInvalidValue;
}

hipError_t launch_max_speed(const KProb& pb, const double* u, double* smax, hipStream_t s) {
  unsigned long long* sm = reinterpret_cast<unsigned long long*>(smax);
  ProfScope ps("max_speed", s);
  k_zero_u64<<<1, 64, 0, s>>>(sm, pb.dim);
  ACAT_CHECK_LAUNCH();
  const int64_t n = pb.nx * (pb.dim == 2 ? pb.ny : 1);
  int64_t blocks = (n + BLOCK - 1) / BLOCK;
  if (blocks > num_cus()) blocks = num_cus();   // one atomic per block: few blocks, many cells each
  const unsigned gb = (unsigned)blocks;
  if (pb.dim == 1) {
    if (pb.flux == EUL) k_max_speed<EUL, 1, 3><<<gb, BLOCK, 0, s>>>(pb, u, sm);
    else if (pb.flux == BURG) k_max_speed<BURG, 1, 1><<<gb, BLOCK, 0, s>>>(pb, u, sm);
    else k_max_speed<ADV, 1, 1><<<gb, BLOCK, 0, s>>>(pb, u, sm);
  } else {
    if (pb.flux == EUL) k_max_speed<EUL, 2, 4><<<gb, BLOCK, 0, s>>>(pb, u, sm);
    else k_max_speed<ADV, 2, 1><<<gb, BLOCK, 0, s>>>(pb, u, sm);
  }
  ACAT_CHECK_LAUNCH();
  return hipSuccess;
}

hipError_t launch_cfl_dt(const KProb& pb, const double* smax, double cfl, double t_final, double* t_dev,
                         double* dt_dev, hipStream_t s) {
  ProfScope ps("cfl_dt", s);
  k_cfl_dt<<<1, 1, 0, s>>>(pb.dim, pb.dx, pb.dy, smax, cfl, t_final, t_dev, dt_dev);
  ACAT_CHECK_LAUNCH();
  return hipSuccess;
}

// Coefficient tables as the kernels use them (host copy of the same constexpr data).
void copy_tables(int p, double* g1, double* gt, double* eta, double* tau) {
  const int n = 2 * p;
  for (int a = 0; a < n; ++a)
    for (int l = 0; l < n; ++l) {
      if (g1) g1[a * n + l] = TB.G1[p][a][l];
      if (gt) gt[a * n + l] = TB.GT[p][a][l];
    }
  for (int a = 0; a < n; ++a) {
    if (eta) eta[a] = TB.ETA[p][a];
    if (tau) tau[a] = TB.TAU[p][a];
  }
}

}  // namespace acat
