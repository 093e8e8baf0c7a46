// The corner recursion of Sec. 4 with four stencil nodes per lane.
//
// A corner of orders (Q1, Q2) has (2 Q1)(2 Q2) nodes; lane (a, b), a < Q1,
// b < Q2, holds the nodes (a, b), (a', b), (a, b'), (a', b') with the mirror
// indices a' = 2 Q1 - 1 - a and b' = 2 Q2 - 1 - b.  A level's spatial
// derivatives read the rows b, b' and the columns a, a' of the exchanged
// fluxes from LDS, each value used for two nodes, where one node per lane
// reads a row and a column for every node: half the LDS reads.  The LDS's
// return rate is what bounds the recursion with one node per lane (a level of
// class (3, 3) reads 24 x 16 B per node, about the time of its 220 FP64
// operations).  The first-derivative weights of a mirror node are the negated
// weights of the node in reverse, so one set serves both.
//
// Corners are packed whole into a wavefront (Q1 Q2 lanes each; 7 corners of
// class (3, 3) in 63 lanes) and exchange in the wave's own LDS, whose
// operations are performed in issue order: no barrier, one buffer.
//
// Only row j2 = 0 of the last level's Fh and column j1 = 0 of its Gh enter the
// fluxes: of a lane's four nodes the last level evaluates one for both fluxes,
// one for F, one for G and skips the fourth.
#pragma once

#include <hip/hip_runtime.h>

#include <utility>

#include "step_common.hpp"

namespace acat {
namespace {

template <int Q1, int Q2>
struct Lanes4 {
  static constexpr int N1 = 2 * Q1, N2 = 2 * Q2, L = Q1 * Q2;
  static constexpr int CPW = 64 / L;                                  // corners per wave
  static constexpr int TOTAL = CPW + (64 % L ? 1 : 0);                // and the idle lanes' spare one
  static constexpr int GS = N1 * N2 + ((N1 * N2) % 8 == 4 ? 1 : 0);   // exchange slots from corner to corner
  static constexpr int STRIDE = TOTAL * GS;                           // slots per plane
};

// Series sums of the corners of a wave: task t of a corner accumulates
// S = sum_k Fh^{k-1} / k! of one node of the row j2 = 0 (DOF), or
// sum_k Gh^{k-1} / k! of one node of the column j1 = 0 (DOG), two components
// each (one for a scalar law), from the exchanged fluxes of every level.
template <int NV, int Q1, int Q2, bool DOF, bool DOG>
struct Series4 {
  using Ln = Lanes4<Q1, Q2>;
  static constexpr int PL = NV == 1 ? 1 : NV / 2, W = NV == 1 ? 1 : 2;
  static constexpr int NF = DOF ? Ln::N1 * PL : 0, NT = NF + (DOG ? Ln::N2 * PL : 0);
  static constexpr int TPL = (Ln::CPW * NT + 63) / 64;   // tasks per lane
  int off[TPL];     // doubles from the exchange's start
  double S[TPL][W];
  __device__ __forceinline__ explicit Series4(int lane) {
#pragma unroll
    for (int s = 0; s < TPL; ++s) {
      int t = lane + 64 * s;
      if (t >= Ln::CPW * NT) t = 0;
      const int g = t / NT;
      t -= g * NT;
      const bool f = DOF && t < NF;
      const int r = f ? t : t - NF, n = f ? Ln::N1 : Ln::N2;
      const int pl = r / n, l = r - pl * n;
      const int slot = g * Ln::GS + (f ? (Q2 - 1) * Ln::N1 + l : l * Ln::N1 + (Q1 - 1));
      off[s] = NV == 1 ? 2 * slot + (f ? 0 : 1) : 2 * (((f ? 0 : PL) + pl) * Ln::STRIDE + slot);
#pragma unroll
      for (int w = 0; w < W; ++w) S[s][w] = 0.0;
    }
  }
  // the term of the exchanged Fh^{k-1}, Gh^{k-1}
  __device__ __forceinline__ void add(const double* x, int k) {
#pragma unroll
    for (int s = 0; s < TPL; ++s)
#pragma unroll
      for (int w = 0; w < W; ++w) S[s][w] = fma(TB.INVFACT[k], x[off[s] + w], S[s][w]);
  }
  // the sums of the wave's corners, NT W doubles per corner
  __device__ __forceinline__ void put(double* sums, int lane) const {
#pragma unroll
    for (int s = 0; s < TPL; ++s) {
      const int t = lane + 64 * s;
      if (t < Ln::CPW * NT) {
#pragma unroll
        for (int w = 0; w < W; ++w) sums[W * t + w] = S[s][w];
      }
    }
  }
  // where component c of node l's F (G) series of corner g is among them
  static __device__ __forceinline__ int at(int g, int c, int l, bool G) {
    return W * (g * NT + (G ? NF : 0) + (c / W) * (G ? Ln::N2 : Ln::N1) + l) + c % W;
  }
};

template <class F, int... K>
__device__ __forceinline__ void for_levels4(F&& f, std::integer_sequence<int, K...>) {
  (f(std::integral_constant<int, K + 2>{}), ...);
}

// One recursion over the rectangle with time nodes J_QT (Taylor order 2 QT);
// nodes n = i + 2 j: i picks a or a', j picks b or b'.  The same operations
// per node, in the same order, as one node per lane.  wx, wy: derivative
// weights of the nodes a (row) and b (column) times -lamx and -lamy; x: the
// wave's exchange planes; slot: of the four nodes; row, col: first slots of
// the rows b, b' and columns a, a'.
template <int FLUX, int NV, int Q1, int Q2, int QT, bool DOF, bool DOG>
__device__ __forceinline__ void corner4_pass(const Phys& ph, const double (&u)[4][NV], const double (&f0)[4][NV],
                                             const double (&g0)[4][NV], const double (&wx)[2 * Q1],
                                             const double (&wy)[2 * Q2], double2* x, const int (&slot)[4],
                                             const int (&row)[2], const int (&col)[2],
                                             Series4<NV, Q1, Q2, DOF, DOG>& ser) {
  using Ln = Lanes4<Q1, Q2>;
  constexpr int N1 = Ln::N1, N2 = Ln::N2, T = 2 * QT;
  const double* xr = reinterpret_cast<const double*>(x);
  double W[T][4][NV];   // Taylor predictions u + sum_{l<kk} r^l/l! U^l at the time nodes r != 0
#pragma unroll
  for (int ri = 0; ri < T; ++ri)
#pragma unroll
    for (int n = 0; n < 4; ++n)
#pragma unroll
      for (int c = 0; c < NV; ++c) W[ri][n][c] = u[n][c];
#pragma unroll
  for (int n = 0; n < 4; ++n) Xch<NV>::put(x, Ln::STRIDE, slot[n], f0[n], g0[n]);
  wave_sync();
  // one recursion level: U^{kk-1} from the exchanged Fh^{kk-2}, Gh^{kk-2};
  // predictions; Fh^{kk-1}, Gh^{kk-1}, exchanged
  auto level = [&](auto kkc) {
    constexpr int kk = decltype(kkc)::value;
    ser.add(xr, kk - 1);
    // U^{kk-1} = -lamx d_x Fh^{kk-2} - lamy d_y Gh^{kk-2}: one chain of fused
    // multiply-adds per node and component over the row (x), then the column (y)
    double Uk[4][NV];
#pragma unroll
    for (int n = 0; n < 4; ++n)
#pragma unroll
      for (int c = 0; c < NV; ++c) Uk[n][c] = 0.0;
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int l = 0; l < N1; ++l)
#pragma unroll
        for (int c = 0; c < NV; ++c) {
          const double v = Xch<NV>::get(xr, Ln::STRIDE, row[j] + l, c, false);
          Uk[2 * j][c] = fma(wx[l], v, Uk[2 * j][c]);
          Uk[2 * j + 1][c] = fma(-wx[N1 - 1 - l], v, Uk[2 * j + 1][c]);
        }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int l = 0; l < N2; ++l)
#pragma unroll
        for (int c = 0; c < NV; ++c) {
          const double v = Xch<NV>::get(xr, Ln::STRIDE, col[i] + l * N1, c, true);
          Uk[i][c] = fma(wy[l], v, Uk[i][c]);
          Uk[i + 2][c] = fma(-wy[N2 - 1 - l], v, Uk[i + 2][c]);
        }
    wave_sync();
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      const bool doF = kk < T || (DOF && n < 2), doG = kk < T || (DOG && n % 2 == 0);
      if (!doF && !doG) continue;
#pragma unroll
      for (int ri = 0; ri < T; ++ri) {
        const int r = ri - QT + 1;
        if (r == 0) continue;
#pragma unroll
        for (int c = 0; c < NV; ++c) W[ri][n][c] = fma(TB.TAYLOR[r + PMAX - 1][kk - 1], Uk[n][c], W[ri][n][c]);
      }
      double nf[NV], ng[NV];
#pragma unroll
      for (int c = 0; c < NV; ++c) {
        nf[c] = 0.0;
        ng[c] = 0.0;
      }
      // Euler: the reciprocal densities of all predicted states first, their
      // refinement steps interleaved
      double rho[T - 1], ir[T - 1];
      if constexpr (FLUX == EUL) {
#pragma unroll
        for (int ri = 0; ri < T; ++ri)
          if (ri != QT - 1) rho[ri < QT - 1 ? ri : ri - 1] = W[ri][n][0];
        recip_n(rho, ir);
      }
#pragma unroll
      for (int ri = 0; ri < T; ++ri) {
        const int r = ri - QT + 1;
        // a time node whose weight is exactly zero adds nothing to Fh, Gh: its
        // fluxes are not evaluated (the same sums for finite values)
        if (TB.GT[QT][kk - 1][ri] == 0.0) continue;
        double pf[NV], pg[NV];
        if (r == 0) {
#pragma unroll
          for (int c = 0; c < NV; ++c) {
            pf[c] = f0[n][c];
            pg[c] = g0[n][c];
          }
        } else if constexpr (FLUX == EUL) {
          euler2d_ir(ph, W[ri][n], ir[ri < QT - 1 ? ri : ri - 1], pf, pg);
        } else {
          flux2d<FLUX, NV>(ph, W[ri][n], pf, pg);
        }
#pragma unroll
        for (int c = 0; c < NV; ++c) {
          if (doF) nf[c] = fma(TB.GT[QT][kk - 1][ri], pf[c], nf[c]);
          if (doG) ng[c] = fma(TB.GT[QT][kk - 1][ri], pg[c], ng[c]);
        }
      }
      Xch<NV>::put(x, Ln::STRIDE, slot[n], nf, ng);
    }
    wave_sync();
  };
  for_levels4(level, std::make_integer_sequence<int, T - 1>{});
  ser.add(xr, T);
  wave_sync();
}

// 2D FL-CAT2 (Sec. 4), component c of the x- (y-, isG) flux of the corner
// (i1, i2): psi^1 CAT2 + (1 - psi^1) F^lo in this direction.
template <int FLUX, int NV>
__device__ __forceinline__ double fl_cat2_2d(const KProb& pb, const KStep& st, double dt, int i1, int i2, bool isG,
                                             int c, double v) {
  const int nx32 = (int)pb.nx, ny32 = (int)pb.ny, ioff = (int)pb.ioff;
  const int64_t nx = pb.nx, ny = pb.ny;
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
  return psi * v + (1.0 - psi) * lo;
}

// Fluxes of the corners of order class (Q1, Q2) in the wave's share `sl` of
// the class list.  SQUARE: list entries carry the square-stencil variant's
// tags (square classes only).  x: the wave's exchange planes in LDS
// (Xch<NV>::NP STRIDE double2).
template <int FLUX, int NV, int Q1, int Q2, bool SQUARE>
__device__ __forceinline__ void corner4_body(const KProb& pb, const KStep& st, const Slice& sl, double2* x) {
  static_assert(Q1 > 1 || Q2 > 1, "class (1,1) runs in k_flux2d_q11");
  using Ln = Lanes4<Q1, Q2>;
  constexpr int N1 = Ln::N1, N2 = Ln::N2;
  const int lane = __lane_id();
  const bool in = lane < Ln::CPW * Ln::L;
  const int g = in ? lane / Ln::L : Ln::CPW;
  const int a = lane % Ln::L % Q1, b = lane % Ln::L / Q1;
  const double dt = step_dt(st);
  const double lamx = dt / pb.dx, lamy = dt / pb.dy;
  const int64_t nx = pb.nx, ny = pb.ny, plane = pb.nx * pb.ny;
  const int nx32 = (int)pb.nx, ny32 = (int)pb.ny, ioff = (int)pb.ioff;
  const uint32_t n1u = (uint32_t)pb.n1;
  double wx[N1], wy[N2];
#pragma unroll
  for (int l = 0; l < N1; ++l) wx[l] = -lamx * TB.G1[Q1][a][l];
#pragma unroll
  for (int l = 0; l < N2; ++l) wy[l] = -lamy * TB.G1[Q2][b][l];
  const int na[2] = {a, N1 - 1 - a}, nb[2] = {b, N2 - 1 - b};
  const int row[2] = {g * Ln::GS + nb[0] * N1, g * Ln::GS + nb[1] * N1};
  const int col[2] = {g * Ln::GS + na[0], g * Ln::GS + na[1]};
  const int slot[4] = {row[0] + na[0], row[0] + na[1], row[1] + na[0], row[1] + na[1]};

  for (int64_t base = sl.lo; base < sl.hi; base += Ln::CPW) {
    const bool valid = in && base + g < sl.hi;
    double u[4][NV], f0[4][NV], g0[4][NV];
    {
      const int32_t raw = valid ? sl.items[base + g] : 0;
      const int32_t e = SQUARE ? (raw & ((1 << LIST_TAG_SHIFT) - 1)) : raw;
      const uint32_t eq = (uint32_t)e / n1u;
      const int i2 = (int)eq + ioff, i1 = (int)((uint32_t)e - eq * n1u) + ioff;
#pragma unroll
      for (int n = 0; n < 4; ++n) {
        const int xx = bc_index32(i1 + (na[n % 2] - Q1 + 1), nx32, pb.bc);
        const int yy = bc_index32(i2 + (nb[n / 2] - Q2 + 1), ny32, pb.bc);
        const double* un = st.u + ((int64_t)yy * nx + xx);
#pragma unroll
        for (int c = 0; c < NV; ++c) u[n][c] = valid ? un[c * plane] : 1.0;
      }
    }
#pragma unroll
    for (int n = 0; n < 4; ++n) flux2d<FLUX, NV>(pb.ph, u[n], f0[n], g0[n]);
    using Both = Series4<NV, Q1, Q2, true, true>;
    using SF = Series4<NV, Q1, Q2, true, false>;
    using SG = Series4<NV, Q1, Q2, false, true>;
    double* sums = reinterpret_cast<double*>(x);
    constexpr int SGOFF = SF::W * SF::NT * Ln::CPW;   // where the G sums of two recursions start
    if constexpr (Q1 == Q2) {
      Both ser(lane);
      corner4_pass<FLUX, NV, Q1, Q2, Q1, true, true>(pb.ph, u, f0, g0, wx, wy, x, slot, row, col, ser);
      ser.put(sums, lane);
    } else {
      SF sf(lane);
      SG sg(lane);
      corner4_pass<FLUX, NV, Q1, Q2, Q1, true, false>(pb.ph, u, f0, g0, wx, wy, x, slot, row, col, sf);
      corner4_pass<FLUX, NV, Q1, Q2, Q2, false, true>(pb.ph, u, f0, g0, wx, wy, x, slot, row, col, sg);
      sf.put(sums, lane);
      sg.put(sums + SGOFF, lane);
    }
    wave_sync();
    // F_c = sum_l eta_l SF_(l,0),c and G_c = sum_l eta_l SG_(0,l),c: 2 NV results per corner
    for (int o = lane; o < Ln::CPW * 2 * NV; o += 64) {
      const int og = o / (2 * NV), oc = o - og * (2 * NV);
      if (base + og >= sl.hi) break;
      const int32_t raw = sl.items[base + og];
      const int32_t e = SQUARE ? (raw & ((1 << LIST_TAG_SHIFT) - 1)) : raw;
      const int tag = SQUARE ? (raw >> LIST_TAG_SHIFT) : 0;   // which flux to store (1 F, 2 G, 0 both)
      const uint32_t eq = (uint32_t)e / n1u;
      const int i2 = (int)eq + ioff, i1 = (int)((uint32_t)e - eq * n1u) + ioff;
      const bool isG = oc >= NV;
      const int c = isG ? oc - NV : oc;
      // transmissive ghost corners need one flux only; tagged entries one flux each
      const bool need = isG ? (i1 >= 0 && tag != 1) : (i2 >= 0 && tag != 2);
      if (!need) continue;
      double v = 0.0;
      if (!isG) {
#pragma unroll
        for (int l = 0; l < N1; ++l)
          v = fma(TB.ETA[Q1][l], sums[Q1 == Q2 ? Both::at(og, c, l, false) : SF::at(og, c, l, false)], v);
      } else {
#pragma unroll
        for (int l = 0; l < N2; ++l)
          v = fma(TB.ETA[Q2][l], sums[Q1 == Q2 ? Both::at(og, c, l, true) : SGOFF + SG::at(og, c, l, true)], v);
      }
      if ((!isG && Q1 == 1) || (isG && Q2 == 1))
        v = fl_cat2_2d<FLUX, NV>(pb, st, dt, i1, i2, isG, c, v);
      if (isG) st.Gy[((int64_t)c * pb.nIy + (i2 - ioff)) * nx + i1] = v;
      else st.Fx[((int64_t)c * ny + i2) * pb.nIx + (i1 - ioff)] = v;
    }
    wave_sync();
  }
}

}  // namespace
}  // namespace acat
