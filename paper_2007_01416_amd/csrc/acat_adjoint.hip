// Adjoint of one ACAT step with frozen decisions (orders, psi^1, Rusanov
// speed, time step): ubar_in = ubar_out + sum over interfaces of
// (dF/du)^T Fbar, with Fbar_k = lambda (ubar_{i+1} - ubar_i) for the
// interface between cells i and i+1 (in 2D likewise for G along y).
//
// Per interface (1D) or corner (2D) the kernels recompute the CAT recursion
// of the forward step (Sec. 2.2; Sec. 4 corner recursion) in registers, one
// lane per stencil node, keeping the Taylor history U^1..U^{2q-1} of the
// node, then run it backwards: flux Jacobian-transpose products at the
// predicted states, and for the spatial derivative of each level the
// transposed row/column sums through LDS.  Each lane writes the
// contribution to its node into a per-item buffer; a gather kernel adds, for
// every cell, the contributions of all items whose stencil covers it in a
// fixed order (deterministic, no atomics).
#include <hip/hip_runtime.h>

#include <utility>

#include "acat_internal.hpp"
#include "coeffs.hpp"
#include "step_common.hpp"

namespace acat {
namespace {

// ======================================================================= 1D
// contribution buffer, slot-major: C[c][slot][k] with slot = j + P - 1 for the
// node at offset j in [-P+1, P] of interface k, so that a gather over one
// offset reads consecutive interfaces
// An interface of order p on the 2p lanes of its group (grp; wave-local): the
// adjoint contributions of interface k at its nodes.  xs: the wave's LDS
// exchange, 2 NV NS doubles.
template <int FLUX, int NV, int p>
struct Adj1D {
  static constexpr int L = 2 * p, SL = L + 1;
  using Grp = Groups<L, 64>;
  static_assert(Grp::WAVE_LOCAL, "the exchange needs no block barrier");
  static constexpr int NS = Grp::TOTAL * SL;
  static constexpr int LDS_DOUBLES = 2 * NV * NS;

  Grp grp;
  double g1[L], g1T[L];   // derivative weights at this lane's node: rows for the recursion, columns for its transpose
  double eta;

  __device__ __forceinline__ explicit Adj1D(int lane) : grp(lane) {
#pragma unroll
    for (int l = 0; l < L; ++l) {
      g1[l] = TB.G1[p][grp.node][l];
      g1T[l] = TB.G1[p][l][grp.node];
    }
    eta = TB.ETA[p][grp.node];
  }
};

template <int FLUX, int NV, int p>
__device__ __forceinline__ void adj1d_body(const KProb& pb, const KStep& st, const Adj1D<FLUX, NV, p>& adj,
                                           bool valid, int32_t k, double dt, const double* __restrict__ ubo,
                                           double* __restrict__ C, double* xs) {
  constexpr int L = 2 * p, SL = Adj1D<FLUX, NV, p>::SL, NS = Adj1D<FLUX, NV, p>::NS;
  const int g = adj.grp.g, a = adj.grp.node;
  const int slot = g * SL + a;
  const double lam = dt / pb.dx;
  const int64_t nx = pb.nx, nI = pb.nIx;
  const int nx32 = (int)nx;
  const int64_t cstride = nI * 2 * pb.P;
  const double(&g1)[L] = adj.g1, (&g1T)[L] = adj.g1T;
  int buf = 0;
  const int i = k + (int)pb.ioff;
  const int node = bc_node32(i, a - p + 1, nx32, pb.bc);
  double u[NV], Fb[NV];
#pragma unroll
  for (int c = 0; c < NV; ++c) u[c] = valid ? st.u[c * nx + node] : 1.0;
  // Fbar = lambda (ubar_{i+1} - ubar_i); a transmissive boundary interface
  // updates only the cell inside the grid
  const bool hasR = valid && (pb.bc == PERIODIC || i + 1 < nx32);
  const bool hasL = valid && i >= 0;
  const int cr = bc_index32(i + 1, nx32, pb.bc), cl = bc_index32(i, nx32, pb.bc);
#pragma unroll
  for (int c = 0; c < NV; ++c) {
    const double ur = hasR ? ubo[c * nx + cr] : 0.0;
    const double ul = hasL ? ubo[c * nx + cl] : 0.0;
    Fb[c] = lam * (ur - ul);
  }
  double psi = 1.0, al = 0.0;
  if constexpr (p == 1) {
    if (valid) {
      psi = st.psix[k];
      al = st.alx[k];
    }
  }
  // ---- forward recomputation, keeping U^l at this node
  double fh0[NV], cur[NV];
  flux1d<FLUX, NV>(pb.ph, u, fh0);
#pragma unroll
  for (int c = 0; c < NV; ++c) cur[c] = fh0[c];
  double U[L][NV];
#pragma unroll
  for (int kk = 2; kk <= 2 * p - 1; ++kk) {   // Fh^{2p-1} is not needed backwards
#pragma unroll
    for (int c = 0; c < NV; ++c) xs[(buf * NV + c) * NS + slot] = cur[c];
    wave_sync();
#pragma unroll
    for (int c = 0; c < NV; ++c) {
      double sacc = 0.0;
#pragma unroll
      for (int l = 0; l < L; ++l) sacc = fma(g1[l], xs[(buf * NV + c) * NS + g * SL + l], sacc);
      U[kk - 1][c] = -lam * sacc;
    }
    buf ^= 1;
    double nxt[NV];
#pragma unroll
    for (int c = 0; c < NV; ++c) nxt[c] = 0.0;
#pragma unroll
    for (int ri = 0; ri < L; ++ri) {
      const int r = ri - p + 1;
      double ph[NV];
      if (r == 0) {
#pragma unroll
        for (int c = 0; c < NV; ++c) ph[c] = fh0[c];
      } else {
        double w[NV];
#pragma unroll
        for (int c = 0; c < NV; ++c) {
          double sacc = u[c];
#pragma unroll
          for (int l = 1; l <= kk - 1; ++l) sacc = fma(TB.TAYLOR[r + PMAX - 1][l], U[l][c], sacc);
          w[c] = sacc;
        }
        flux1d<FLUX, NV>(pb.ph, w, ph);
      }
#pragma unroll
      for (int c = 0; c < NV; ++c) nxt[c] = fma(TB.GT[p][kk - 1][ri], ph[c], nxt[c]);
    }
#pragma unroll
    for (int c = 0; c < NV; ++c) cur[c] = nxt[c];
  }
  // U^{2p-1}
  if (2 * p >= 2) {
#pragma unroll
    for (int c = 0; c < NV; ++c) xs[(buf * NV + c) * NS + slot] = cur[c];
    wave_sync();
#pragma unroll
    for (int c = 0; c < NV; ++c) {
      double sacc = 0.0;
#pragma unroll
      for (int l = 0; l < L; ++l) sacc = fma(g1[l], xs[(buf * NV + c) * NS + g * SL + l], sacc);
      U[2 * p - 1][c] = -lam * sacc;
    }
    buf ^= 1;
  }
  // ---- reverse sweep
  // F = sum_j eta_j S_j, S_j = sum_k Fh^{k-1}_j / k!  =>  Sbar_j = eta_j psi Fbar
  double sb[NV], ub[NV], f0b[NV], fhb[NV];
#pragma unroll
  for (int c = 0; c < NV; ++c) {
    sb[c] = adj.eta * psi * Fb[c];
    ub[c] = 0.0;
    f0b[c] = 0.0;
    fhb[c] = TB.INVFACT[2 * p] * sb[c];   // Fhbar^{2p-1}
  }
  double Ub[L][NV];
#pragma unroll
  for (int l = 0; l < L; ++l)
#pragma unroll
    for (int c = 0; c < NV; ++c) Ub[l][c] = 0.0;
#pragma unroll
  for (int kk = 2 * p; kk >= 2; --kk) {
    // as in the 2D recursion: not the forward sweep's predicted states, held from
    // there to here (registers and scratch of p = 3, 4, 5 in a kernel of its own: 352,
    // 512 + 472 bytes, 512 + 2180; so 270, 440, 512 + 488).  A scalar's fit up to
    // p = 6 (Burgers 2e5 cells, all orders by tiles: P = 4 94 us, opaque 88; P = 5 159,
    // 164; P = 6 402, 411).
    if constexpr (p >= 2 && (NV > 1 || p <= 4)) {
#pragma unroll
      for (int l = 1; l <= kk - 1; ++l)
#pragma unroll
        for (int c = 0; c < NV; ++c) asm volatile("" : "+v"(U[l][c]));
    }
    // Fh^{kk-1} = sum_r GT_r phi_r
#pragma unroll
    for (int ri = 0; ri < L; ++ri) {
      const int r = ri - p + 1;
      double phb[NV];
#pragma unroll
      for (int c = 0; c < NV; ++c) phb[c] = TB.GT[p][kk - 1][ri] * fhb[c];
      if (r == 0) {
#pragma unroll
        for (int c = 0; c < NV; ++c) f0b[c] += phb[c];
      } else {
        double w[NV], wb[NV];
#pragma unroll
        for (int c = 0; c < NV; ++c) {
          double sacc = u[c];
#pragma unroll
          for (int l = 1; l <= kk - 1; ++l) sacc = fma(TB.TAYLOR[r + PMAX - 1][l], U[l][c], sacc);
          w[c] = sacc;
          wb[c] = 0.0;
        }
        flux1d_vjp<FLUX, NV>(pb.ph, w, phb, wb);
#pragma unroll
        for (int c = 0; c < NV; ++c) {
          ub[c] += wb[c];
#pragma unroll
          for (int l = 1; l <= kk - 1; ++l) Ub[l][c] += TB.TAYLOR[r + PMAX - 1][l] * wb[c];
        }
      }
    }
    // U^{kk-1}_a = -lam sum_l g1[a][l] Fh^{kk-2}_l  =>  Fhbar^{kk-2}_a += -lam sum_j g1[j][a] Ubar_j
#pragma unroll
    for (int c = 0; c < NV; ++c) xs[(buf * NV + c) * NS + slot] = Ub[kk - 1][c];
    wave_sync();
#pragma unroll
    for (int c = 0; c < NV; ++c) {
      double sacc = 0.0;
#pragma unroll
      for (int j = 0; j < L; ++j) sacc += g1T[j] * xs[(buf * NV + c) * NS + g * SL + j];
      fhb[c] = TB.INVFACT[kk - 1] * sb[c] - lam * sacc;   // Fhbar^{kk-2}
    }
    buf ^= 1;
  }
  // Fh^0 = f(u) also enters every r = 0 term
#pragma unroll
  for (int c = 0; c < NV; ++c) f0b[c] += fhb[c];
  flux1d_vjp<FLUX, NV>(pb.ph, u, f0b, ub);
  if constexpr (p == 1) {
    // Rusanov part of the FL-CAT2 blend: (1 - psi) [(f_i + f_{i+1})/2 - alpha/2 (u_{i+1} - u_i)]
    double lb[NV], zero[NV];
#pragma unroll
    for (int c = 0; c < NV; ++c) {
      lb[c] = 0.5 * (1.0 - psi) * Fb[c];
      zero[c] = 0.0;
    }
    flux1d_vjp<FLUX, NV>(pb.ph, u, lb, zero);
    const double sp = (pb.flags & FLAG_FLO_LF) ? pb.dx / ((double)pb.dim * dt) : al;
#pragma unroll
    for (int c = 0; c < NV; ++c) ub[c] += zero[c] + (a == 0 ? sp : -sp) * lb[c];
  }
  if (valid) {
#pragma unroll
    for (int c = 0; c < NV; ++c) C[c * cstride + (int64_t)(a - p + pb.P) * nI + k] = ub[c];
  }
}

// ubar_in[m] = ubar_out[m] + the contributions of every interface with a
// stencil node at cell m (through the boundary map), interfaces in
// increasing order, nodes in increasing order.  Periodic: interfaces
// i = m - j, j in [-P+1, P] (node j of interface i is cell m exactly when
// i + j = m, as nx >= 2P).  Transmissive: the same window, extended to the
// first (last) interface for the P cells next to the left (right) edge,
// whose clamped nodes reach them.
template <int NV, int P>
__global__ __launch_bounds__(BLOCK) void k_gather1d(KProb pb, KStep st, const double* __restrict__ ubo,
                                                    const double* __restrict__ C, double* ubi) {
  const int m = blockIdx.x * BLOCK + threadIdx.x;
  const int nx = (int)pb.nx, ioff = (int)pb.ioff, nI = (int)pb.nIx;
  if (m >= nx) return;
  const int64_t cstride = (int64_t)nI * 2 * P;
  const bool per = pb.bc == PERIODIC;
  double acc[NV];
#pragma unroll
  for (int c = 0; c < NV; ++c) acc[c] = ubo[c * pb.nx + m];
  if (per || (m >= P && m < nx - P)) {
    // cell m is node j = m - i of interface i alone
#pragma unroll
    for (int j = P; j >= -P + 1; --j) {
      const int k = bc_node32(m, -j, nx, PERIODIC) - ioff;   // transmissive: an interior cell, nothing wraps
      const int q = st.cls[k] + 1;
      if (j > q || j <= -q) continue;
#pragma unroll
      for (int c = 0; c < NV; ++c) acc[c] += C[c * cstride + (int64_t)(j + P - 1) * nI + k];
    }
  } else {
    const int ilo = m < P ? ioff : m - P;
    const int ihi = m >= nx - P ? nx - 1 : m + P - 1;
    for (int i = ilo; i <= ihi; ++i) {
      const int q = min(st.cls[i - ioff] + 1, P);   // no order beyond P, whatever the map holds
      for (int a = 0; a < 2 * q; ++a) {
        const int j = a - q + 1;
        if (bc_node32(i, j, nx, pb.bc) != m) continue;
#pragma unroll
        for (int c = 0; c < NV; ++c) acc[c] += C[c * cstride + (int64_t)(j + P - 1) * nI + (i - ioff)];
      }
    }
  }
#pragma unroll
  for (int c = 0; c < NV; ++c) ubi[c * pb.nx + m] = acc[c];
}

// ======================================================================= 2D
// One corner recursion forward (keeping U), then backwards.  sfb/sgb: the
// adjoints of this node's series SF / SG; ub accumulates the adjoint of u,
// f0b/g0b those of f(u), g(u).
template <int FLUX, int NV, int Q1, int Q2, int QT>
__device__ __forceinline__ void corner_adjoint(const Phys& ph, const double (&u)[NV],
                                               const double (&f0)[NV], const double (&g0)[NV],
                                               const double* gx, const double* gy,
                                               double2* xsb0, double2* xsb1, int stride, int& buf, int slot,
                                               int gbase, int a1, int a2, const double (&sfb)[NV],
                                               const double (&sgb)[NV], double (&ub)[NV], double (&f0b)[NV],
                                               double (&g0b)[NV]) {
  constexpr int N1 = 2 * Q1, N2 = 2 * Q2, T = 2 * QT;
  double fc[NV], gc[NV];
#pragma unroll
  for (int c = 0; c < NV; ++c) {
    fc[c] = f0[c];
    gc[c] = g0[c];
  }
  double U[T][NV];
  // this node's derivative weights of the forward differences, in registers
  // for the pass (the transposed ones are read from LDS at each use)
  double wfx[N1], wfy[N2];
#pragma unroll
  for (int l = 0; l < N1; ++l) wfx[l] = gx[a1 * N1 + l];
#pragma unroll
  for (int l = 0; l < N2; ++l) wfy[l] = gy[a2 * N2 + l];
  // forward: U^1 .. U^{T-1}
#pragma unroll
  for (int kk = 2; kk <= T; ++kk) {
    double2* xsw = buf ? xsb1 : xsb0;
    Xch<NV>::put(xsw, stride, slot, fc, gc);
    Groups<(2 * Q1) * (2 * Q2)>::sync();
    const double* xr = reinterpret_cast<const double*>(xsw);
    // U^{kk-1} as the forward step forms it: one chain over the row, then
    // the column, with the weights -lamx gamma and -lamy gamma
#pragma unroll
    for (int c = 0; c < NV; ++c) {
      double s = 0.0;
#pragma unroll
      for (int l = 0; l < N1; ++l) s = fma(wfx[l], Xch<NV>::get(xr, stride, gbase + a2 * N1 + l, c, false), s);
#pragma unroll
      for (int l = 0; l < N2; ++l) s = fma(wfy[l], Xch<NV>::get(xr, stride, gbase + l * N1 + a1, c, true), s);
      U[kk - 1][c] = s;
    }
    buf ^= 1;
    if (kk == T) break;
    double nf[NV], ng[NV];
#pragma unroll
    for (int c = 0; c < NV; ++c) {
      nf[c] = 0.0;
      ng[c] = 0.0;
    }
#pragma unroll
    for (int ri = 0; ri < T; ++ri) {
      const int r = ri - QT + 1;
      double pf[NV], pg[NV];
      if (r == 0) {
#pragma unroll
        for (int c = 0; c < NV; ++c) {
          pf[c] = f0[c];
          pg[c] = g0[c];
        }
      } else {
        double w[NV];
#pragma unroll
        for (int c = 0; c < NV; ++c) {
          double sacc = u[c];
#pragma unroll
          for (int l = 1; l <= kk - 1; ++l) sacc = fma(TB.TAYLOR[r + PMAX - 1][l], U[l][c], sacc);
          w[c] = sacc;
        }
        flux2d<FLUX, NV>(ph, w, pf, pg);
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
    }
  }
  // backward
  double fhb[NV], ghb[NV];
#pragma unroll
  for (int c = 0; c < NV; ++c) {
    fhb[c] = TB.INVFACT[T] * sfb[c];
    ghb[c] = TB.INVFACT[T] * sgb[c];
  }
  double Ub[T][NV];
#pragma unroll
  for (int l = 0; l < T; ++l)
#pragma unroll
    for (int c = 0; c < NV; ++c) Ub[l][c] = 0.0;
#pragma unroll
  for (int kk = T; kk >= 2; --kk) {
    // The predicted states below recompute the forward sweep's with the same
    // operations; made opaque, U keeps the compiler from holding those of all
    // levels from there to here instead (up to 4 T^2 doubles; q44: 1112 bytes of
    // scratch per lane, with this 472; P = 3 rectangles with an order 3 in one
    // kernel: 266 spills, then 175; Euler 192^2: 126 us, then 113; the whole P = 4
    // adjoint step of 256^2: 1998 us, then 1377).  At T = 4
    // they fit, and recomputing them costs more: 512^2 P = 2 100.5 us, 104 so.  A scalar
    // law's fit at every T (advection 600^2 q44: 1325 us, opaque 1493).
    if constexpr (T > 4 && NV > 1) {
#pragma unroll
      for (int l = 1; l <= kk - 1; ++l)
#pragma unroll
        for (int c = 0; c < NV; ++c) asm volatile("" : "+v"(U[l][c]));
    }
#pragma unroll
    for (int ri = 0; ri < T; ++ri) {
      const int r = ri - QT + 1;
      double pfb[NV], pgb[NV];
#pragma unroll
      for (int c = 0; c < NV; ++c) {
        pfb[c] = TB.GT[QT][kk - 1][ri] * fhb[c];
        pgb[c] = TB.GT[QT][kk - 1][ri] * ghb[c];
      }
      if (r == 0) {
#pragma unroll
        for (int c = 0; c < NV; ++c) {
          f0b[c] += pfb[c];
          g0b[c] += pgb[c];
        }
      } else {
        double w[NV], wb[NV];
#pragma unroll
        for (int c = 0; c < NV; ++c) {
          double sacc = u[c];
#pragma unroll
          for (int l = 1; l <= kk - 1; ++l) sacc = fma(TB.TAYLOR[r + PMAX - 1][l], U[l][c], sacc);
          w[c] = sacc;
          wb[c] = 0.0;
        }
        flux2d_vjp<FLUX, NV>(ph, w, pfb, pgb, wb);
#pragma unroll
        for (int c = 0; c < NV; ++c) {
          ub[c] += wb[c];
#pragma unroll
          for (int l = 1; l <= kk - 1; ++l) Ub[l][c] += TB.TAYLOR[r + PMAX - 1][l] * wb[c];
        }
      }
    }
    // U^{kk-1} = sum_l wx[a1][l] Fh_(l,a2) + sum_l wy[a2][l] Gh_(a1,l)
    // (wx = -lamx gamma, wy = -lamy gamma)
    //  => Fhbar_(a1,a2) += sum_j wx[j][a1] Ubar_(j,a2); Ghbar likewise along the column
    double2* xsw = buf ? xsb1 : xsb0;
    Xch<NV>::put(xsw, stride, slot, Ub[kk - 1], Ub[kk - 1]);
    Groups<(2 * Q1) * (2 * Q2)>::sync();
    const double* xr = reinterpret_cast<const double*>(xsw);
#pragma unroll
    for (int c = 0; c < NV; ++c) {
      double sx = TB.INVFACT[kk - 1] * sfb[c], sy = TB.INVFACT[kk - 1] * sgb[c];
#pragma unroll
      for (int j = 0; j < N1; ++j) sx = fma(gx[j * N1 + a1], Xch<NV>::get(xr, stride, gbase + a2 * N1 + j, c, false), sx);
#pragma unroll
      for (int j = 0; j < N2; ++j) sy = fma(gy[j * N2 + a2], Xch<NV>::get(xr, stride, gbase + j * N1 + a1, c, true), sy);
      fhb[c] = sx;
      ghb[c] = sy;
    }
    buf ^= 1;
  }
#pragma unroll
  for (int c = 0; c < NV; ++c) {
    f0b[c] += fhb[c];
    g0b[c] += ghb[c];
  }
}

// contribution buffer, slot-major: C[c][slot][e], slot = (j2 + P - 1) 2P + (j1 + P - 1)
// for the node at offset (j1, j2) of corner e (a gather over one offset reads
// consecutive corners)
// PASSES (corners with q1 != q2): 1 = the F recursion only, 2 = the G recursion
// only, added to the contributions the first launch wrote, 3 = both.
// The body runs the items [base, end) of the class's list; xsm: the two LDS
// exchange buffers (2 Xch<NV>::NP adj_stride<L>() double2), gx, gy: LDS, the
// derivative weights times -lamx and -lamy ((2 Q1)^2 and (2 Q2)^2 doubles,
// row-major: rows for the recursion, columns for its transpose).
template <int L>
constexpr int adj_stride() {
  return Groups<L>::WAVE_LOCAL ? Groups<L>::TOTAL * L : BLOCK + L;
}

template <int FLUX, int NV, int Q1, int Q2, int PASSES>
__device__ __forceinline__ void adj2d_body(const KProb& pb, const KStep& st, int tid, double dt,
                                           const int32_t* items, int64_t base, int64_t end,
                                           const double* __restrict__ ubo, double* __restrict__ C, int LMAX,
                                           double2* xsm, const double* gx, const double* gy) {
  constexpr int N1 = 2 * Q1, N2 = 2 * Q2, L = N1 * N2;
  using Grp = Groups<L>;
  constexpr int CPB = Grp::PER_BLOCK;
  constexpr int NP = Xch<NV>::NP;
  constexpr int STRIDE = adj_stride<L>();
  double2* const xs[2] = {xsm, xsm + NP * STRIDE};

  const Grp grp(tid);
  const int g = grp.g;
  const int nd = grp.node;
  const int a1 = nd % N1, a2 = nd / N1;
  const bool inblk = grp.in;
  const double lamx = dt / pb.dx, lamy = dt / pb.dy;
  const int64_t nx = pb.nx, plane = pb.nx * pb.ny;
  const int nx32 = (int)pb.nx, ny32 = (int)pb.ny, ioff = (int)pb.ioff;
  const uint32_t n1u = (uint32_t)pb.n1;
  const int64_t nitems = pb.n1 * pb.n2;
  const int64_t cstride = nitems * LMAX;

  const bool on_row = a2 == Q2 - 1, on_col = a1 == Q1 - 1;

  int buf = 0;
  for (; base < end; base += CPB) {
    const bool valid = inblk && base + g < end;
    const int32_t e = valid ? items[base + g] : 0;
    const uint32_t eq = (uint32_t)e / n1u;
    const int i2 = (int)eq + ioff, i1 = (int)((uint32_t)e - eq * n1u) + ioff;
    const int x = bc_index32(i1 + (a1 - Q1 + 1), nx32, pb.bc);
    const int y = bc_index32(i2 + (a2 - Q2 + 1), ny32, pb.bc);
    double u[NV];
#pragma unroll
    for (int c = 0; c < NV; ++c) u[c] = valid ? st.u[c * plane + (int64_t)y * nx + x] : 1.0;
    // Fbar = lamx (ubar_{i+e1} - ubar_i), Gbar = lamy (ubar_{i+e2} - ubar_i), the
    // terms of cells outside a transmissive grid dropped (an edge flux enters
    // one cell only); corners on the ghost row carry no x-flux, those on the
    // ghost column no y-flux
    const bool per = pb.bc == PERIODIC;
    const bool hasF = valid && i2 >= 0, hasG = valid && i1 >= 0;
    double Fb[NV], Gb[NV];
    {
      const bool in1 = per || i1 >= 0, inr1 = per || i1 + 1 < nx32;
      const bool in2 = per || i2 >= 0, inr2 = per || i2 + 1 < ny32;
      const int x0 = bc_index32(i1, nx32, pb.bc), y0 = bc_index32(i2, ny32, pb.bc);
      const int xr = bc_index32(i1 + 1, nx32, pb.bc), yr = bc_index32(i2 + 1, ny32, pb.bc);
#pragma unroll
      for (int c = 0; c < NV; ++c) {
        const double u0 = valid ? ubo[c * plane + (int64_t)y0 * nx + x0] : 0.0;
        const double ux = valid ? ubo[c * plane + (int64_t)y0 * nx + xr] : 0.0;
        const double uy = valid ? ubo[c * plane + (int64_t)yr * nx + x0] : 0.0;
        Fb[c] = hasF ? lamx * ((inr1 ? ux : 0.0) - (in1 ? u0 : 0.0)) : 0.0;
        Gb[c] = hasG ? lamy * ((inr2 ? uy : 0.0) - (in2 ? u0 : 0.0)) : 0.0;
      }
    }
    double psix = 1.0, alx = 0.0, psiy = 1.0, aly = 0.0;
    if (valid) {
      if (Q1 == 1 && hasF) {
        const int64_t ex = (int64_t)i2 * pb.nIx + (i1 - ioff);
        psix = st.psix[ex];
        alx = st.alx[ex];
      }
      if (Q2 == 1 && hasG) {
        const int64_t ey = (int64_t)(i2 - ioff) * nx + i1;
        psiy = st.psiy[ey];
        aly = st.aly[ey];
      }
    }
    double f0[NV], g0[NV];
    flux2d<FLUX, NV>(pb.ph, u, f0, g0);
    double sfb[NV], sgb[NV], zero[NV], ub[NV], f0b[NV], g0b[NV];
#pragma unroll
    for (int c = 0; c < NV; ++c) {
      sfb[c] = on_row ? TB.ETA[Q1][a1] * psix * Fb[c] : 0.0;
      sgb[c] = on_col ? TB.ETA[Q2][a2] * psiy * Gb[c] : 0.0;
      zero[c] = 0.0;
      ub[c] = 0.0;
      f0b[c] = 0.0;
      g0b[c] = 0.0;
    }
    const int slot = g * L + nd;
    if constexpr (Q1 == Q2) {
      corner_adjoint<FLUX, NV, Q1, Q2, Q1>(pb.ph, u, f0, g0, gx, gy, xs[0], xs[1], STRIDE, buf, slot,
                                           g * L, a1, a2, sfb, sgb, ub, f0b, g0b);
    } else {
      if constexpr ((PASSES & 1) != 0)
        corner_adjoint<FLUX, NV, Q1, Q2, Q1>(pb.ph, u, f0, g0, gx, gy, xs[0], xs[1], STRIDE, buf, slot,
                                             g * L, a1, a2, sfb, zero, ub, f0b, g0b);
      if constexpr ((PASSES & 2) != 0)
        corner_adjoint<FLUX, NV, Q1, Q2, Q2>(pb.ph, u, f0, g0, gx, gy, xs[0], xs[1], STRIDE, buf, slot,
                                             g * L, a1, a2, zero, sgb, ub, f0b, g0b);
    }
    // first-order parts (Rusanov or Lax-Friedrichs) of the FL-CAT2 blends, on
    // the two nodes each one reads
    if (pb.flags & FLAG_FLO_LF) {
      alx = pb.dx / ((double)pb.dim * dt);
      aly = pb.dy / ((double)pb.dim * dt);
    }
    if ((PASSES & 1) != 0 && Q1 == 1 && on_row && (a1 == Q1 - 1 || a1 == Q1)) {
#pragma unroll
      for (int c = 0; c < NV; ++c) {
        const double lb = 0.5 * (1.0 - psix) * Fb[c];
        f0b[c] += lb;
        ub[c] += (a1 == Q1 - 1 ? alx : -alx) * lb;
      }
    }
    if ((PASSES & 2) != 0 && Q2 == 1 && on_col && (a2 == Q2 - 1 || a2 == Q2)) {
#pragma unroll
      for (int c = 0; c < NV; ++c) {
        const double lb = 0.5 * (1.0 - psiy) * Gb[c];
        g0b[c] += lb;
        ub[c] += (a2 == Q2 - 1 ? aly : -aly) * lb;
      }
    }
    flux2d_vjp<FLUX, NV>(pb.ph, u, f0b, g0b, ub);
    const int cslot = (a2 - Q2 + pb.P) * (2 * pb.P) + (a1 - Q1 + pb.P);
    if (valid) {
#pragma unroll
      for (int c = 0; c < NV; ++c) {
        double* dst = C + c * cstride + (int64_t)cslot * nitems + e;
        *dst = PASSES == 2 ? *dst + ub[c] : ub[c];
      }
    }
  }
}

// One class: stages its derivative weights in g1s, then runs a share of its list.
template <int FLUX, int NV, int Q1, int Q2, int PASSES>
__device__ __forceinline__ void adj2d_class(const KProb& pb, const KStep& st, const Slice& sl,
                                            const double* __restrict__ ubo, double* __restrict__ C, int LMAX,
                                            double2* xsm, double* g1s) {
  constexpr int N1 = 2 * Q1, N2 = 2 * Q2;
  const double dt = step_dt(st);
  const double lamx = dt / pb.dx, lamy = dt / pb.dy;
  for (int i = threadIdx.x; i < N1 * N1 + N2 * N2; i += BLOCK)
    g1s[i] = i < N1 * N1 ? -lamx * TB.G1[Q1][i / N1][i % N1]
                         : -lamy * TB.G1[Q2][(i - N1 * N1) / N2][(i - N1 * N1) % N2];
  __syncthreads();
  adj2d_body<FLUX, NV, Q1, Q2, PASSES>(pb, st, (int)threadIdx.x, dt, sl.items, sl.lo, sl.hi, ubo, C, LMAX, xsm, g1s,
                                       g1s + N1 * N1);
}

template <int FLUX, int NV, int Q1, int Q2, int PASSES = 3>
__global__ __launch_bounds__(BLOCK) void k_adj2d(KProb pb, KStep st, const double* __restrict__ ubo,
                                                 double* __restrict__ C, int LMAX) {
  constexpr int L = (2 * Q1) * (2 * Q2);
  __shared__ double2 xsm[2 * Xch<NV>::NP * adj_stride<L>()];
  __shared__ double g1s[(2 * Q1) * (2 * Q1) + (2 * Q2) * (2 * Q2)];
  adj2d_class<FLUX, NV, Q1, Q2, PASSES>(
      pb, st, Slice(st.counts, st.list, (Q1 - 1) * pb.P + (Q2 - 1), Groups<L>::PER_BLOCK), ubo, C, LMAX, xsm, g1s);
}

// Order class (1,1) with ONE LANE PER CORNER: the adjoint of the one-lane
// forward kernel.  The lane holds the corner's four nodes (j1, j2) in
// {0,1}^2 and runs the same reverse sweep as the node-per-lane kernel
// (recursion level 2 backwards, the transposed centred differences, the
// blends' first-order parts, the Jacobian-transpose products), skipping
// the terms that are zero for this class: the predicted-state adjoint at
// node (1,1), which no flux reads.  Writes the four nodes' contributions.
template <int FLUX, int NV>
__device__ __forceinline__ void adj2d_q11(const KProb& pb, const KStep& st, int tid, double dt, const int32_t* items,
                                          int64_t base, int64_t end, const double* __restrict__ ubo,
                                          double* __restrict__ C, int LMAX) {
  const double lamx = dt / pb.dx, lamy = dt / pb.dy;
  double gx[2][2], gy[2][2];   // -lamx G1[1][a][l], -lamy G1[1][a][l]
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int l = 0; l < 2; ++l) {
      gx[a][l] = -lamx * TB.G1[1][a][l];
      gy[a][l] = -lamy * TB.G1[1][a][l];
    }
  const double tay = TB.TAYLOR[PMAX][1];
  const double gt0 = TB.GT[1][1][0], gt1 = TB.GT[1][1][1];
  const int64_t nx = pb.nx, plane = pb.nx * pb.ny;
  const int nx32 = (int)pb.nx, ny32 = (int)pb.ny, ioff = (int)pb.ioff;
  const uint32_t n1u = (uint32_t)pb.n1;
  const int64_t nitems = pb.n1 * pb.n2;
  const int64_t cstride = nitems * LMAX;
  const bool per = pb.bc == PERIODIC;
  for (int64_t it = base + tid; it < end; it += BLOCK) {
    const int32_t e = items[it];
    const uint32_t eq = (uint32_t)e / n1u;
    const int i2 = (int)eq + ioff, i1 = (int)((uint32_t)e - eq * n1u) + ioff;
    int xs[2], ys[2];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      xs[a] = bc_index32(i1 + a, nx32, pb.bc);
      ys[a] = bc_index32(i2 + a, ny32, pb.bc);
    }
    // Fbar = lamx (ubar_{i+e1} - ubar_i), Gbar = lamy (ubar_{i+e2} - ubar_i);
    // ghost-row corners carry no x-flux, ghost-column corners no y-flux
    const bool hasF = i2 >= 0, hasG = i1 >= 0;
    double Fb[NV], Gb[NV];
    {
      const bool in1 = per || i1 >= 0, inr1 = per || i1 + 1 < nx32;
      const bool in2 = per || i2 >= 0, inr2 = per || i2 + 1 < ny32;
#pragma unroll
      for (int c = 0; c < NV; ++c) {
        const double u0 = ubo[c * plane + (int64_t)ys[0] * nx + xs[0]];
        const double ux = ubo[c * plane + (int64_t)ys[0] * nx + xs[1]];
        const double uy = ubo[c * plane + (int64_t)ys[1] * nx + xs[0]];
        Fb[c] = hasF ? lamx * ((inr1 ? ux : 0.0) - (in1 ? u0 : 0.0)) : 0.0;
        Gb[c] = hasG ? lamy * ((inr2 ? uy : 0.0) - (in2 ? u0 : 0.0)) : 0.0;
      }
    }
    double psix = 1.0, alx = 0.0, psiy = 1.0, aly = 0.0;
    if (hasF) {
      const int64_t ex = (int64_t)i2 * pb.nIx + (i1 - ioff);
      psix = st.psix[ex];
      alx = st.alx[ex];
    }
    if (hasG) {
      const int64_t ey = (int64_t)(i2 - ioff) * nx + i1;
      psiy = st.psiy[ey];
      aly = st.aly[ey];
    }
    if (pb.flags & FLAG_FLO_LF) {
      alx = pb.dx / ((double)pb.dim * dt);
      aly = pb.dy / ((double)pb.dim * dt);
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
    // adjoints: ub of the node states, f0b/g0b of the point fluxes, Ub1 of U^1
    double ub[2][2][NV], f0b[2][2][NV], g0b[2][2][NV], Ub1[2][2][NV];
    // series adjoints: sfb on the row j2 = 0, sgb on the column j1 = 0
    double sfb[2][NV], sgb[2][NV];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int c = 0; c < NV; ++c) {
        sfb[a][c] = TB.ETA[1][a] * psix * Fb[c];
        sgb[a][c] = TB.ETA[1][a] * psiy * Gb[c];
      }
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int c = 0; c < NV; ++c) {
          // level 2 backwards, time node r = 0: the point fluxes' share
          const double fhb = (b == 0) ? TB.INVFACT[2] * sfb[a][c] : 0.0;
          const double ghb = (a == 0) ? TB.INVFACT[2] * sgb[b][c] : 0.0;
          f0b[b][a][c] = gt0 * fhb;
          g0b[b][a][c] = gt0 * ghb;
          ub[b][a][c] = 0.0;
          Ub1[b][a][c] = 0.0;
        }
    // time node r = 1 at the row and column nodes: the prediction
    // w = u + tay U^1, the flux Jacobians' transpose at w
#pragma unroll
    for (int n = 0; n < 3; ++n) {
      const int a = n == 1 ? 1 : 0, b = n == 2 ? 1 : 0;
      double w[NV], pfb[NV], pgb[NV], wb[NV];
#pragma unroll
      for (int c = 0; c < NV; ++c) {
        double s = 0.0;
        s = fma(gx[a][0], f0[b][0][c], s);
        s = fma(gx[a][1], f0[b][1][c], s);
        s = fma(gy[b][0], g0[0][a][c], s);
        s = fma(gy[b][1], g0[1][a][c], s);
        w[c] = fma(tay, s, u[b][a][c]);
        pfb[c] = (b == 0) ? gt1 * (TB.INVFACT[2] * sfb[a][c]) : 0.0;
        pgb[c] = (a == 0) ? gt1 * (TB.INVFACT[2] * sgb[b][c]) : 0.0;
        wb[c] = 0.0;
      }
      flux2d_vjp<FLUX, NV>(pb.ph, w, pfb, pgb, wb);
#pragma unroll
      for (int c = 0; c < NV; ++c) {
        ub[b][a][c] += wb[c];
        Ub1[b][a][c] = tay * wb[c];
      }
    }
    // U^1 = sum_l gx[a1][l] Fh_(l,a2) + sum_l gy[a2][l] Gh_(a1,l) transposed:
    // Fh^0bar_(a1,a2) = Fh^0 series term + sum_j gx[j][a1] Ub1_(j,a2), and
    // Gh^0bar along the column
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int c = 0; c < NV; ++c) {
          double sx = (b == 0) ? TB.INVFACT[1] * sfb[a][c] : 0.0;
          double sy = (a == 0) ? TB.INVFACT[1] * sgb[b][c] : 0.0;
          sx = fma(gx[0][a], Ub1[b][0][c], sx);
          sx = fma(gx[1][a], Ub1[b][1][c], sx);
          sy = fma(gy[0][b], Ub1[0][a][c], sy);
          sy = fma(gy[1][b], Ub1[1][a][c], sy);
          f0b[b][a][c] += sx;
          g0b[b][a][c] += sy;
        }
    // first-order parts of the FL-CAT2 blends on the two nodes each reads:
    // x on (0,0), (1,0); y on (0,0), (0,1)
#pragma unroll
    for (int c = 0; c < NV; ++c) {
      const double lx = 0.5 * (1.0 - psix) * Fb[c];
      f0b[0][0][c] += lx;
      ub[0][0][c] += alx * lx;
      f0b[0][1][c] += lx;
      ub[0][1][c] += -alx * lx;
      const double ly = 0.5 * (1.0 - psiy) * Gb[c];
      g0b[0][0][c] += ly;
      ub[0][0][c] += aly * ly;
      g0b[1][0][c] += ly;
      ub[1][0][c] += -aly * ly;
    }
    // Jacobian-transpose products at the node states; contributions
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        flux2d_vjp<FLUX, NV>(pb.ph, u[b][a], f0b[b][a], g0b[b][a], ub[b][a]);
        const int cslot = (b - 1 + pb.P) * (2 * pb.P) + (a - 1 + pb.P);
#pragma unroll
        for (int c = 0; c < NV; ++c) C[c * cstride + (int64_t)cslot * nitems + e] = ub[b][a][c];
      }
  }
}

template <int FLUX, int NV>
__global__ __launch_bounds__(BLOCK) void k_adj2d_q11(KProb pb, KStep st, const double* __restrict__ ubo,
                                                     double* __restrict__ C, int LMAX) {
  const Slice sl(st.counts, st.list, 0, BLOCK);
  adj2d_q11<FLUX, NV>(pb, st, (int)threadIdx.x, step_dt(st), sl.items, sl.lo, sl.hi, ubo, C, LMAX);
}

// The mirror classes (QA, QB) and (QB, QA), QA < QB, in one launch (both
// recursions in one pass): the grid is cut into two runs of whole XCD groups
// of blocks sized by the classes' corner counts, at least one per class with
// corners; each block runs its class's body over its share of the list.
// The (1,2) pair is held to two waves per SIMD: unbounded it takes 264
// registers (one wave); bounded, 9 spill to scratch, and it runs 6 % faster.
template <int FLUX, int NV, int QA, int QB>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu((QB <= 2) ? 2 : 1))) void k_adj2d_pair(
    KProb pb, KStep st, const double* __restrict__ ubo, double* __restrict__ C, int LMAX) {
  constexpr int L = (2 * QA) * (2 * QB), CPB = Groups<L>::PER_BLOCK;
  __shared__ double2 xsm[2 * Xch<NV>::NP * adj_stride<L>()];
  __shared__ double g1s[(2 * QA) * (2 * QA) + (2 * QB) * (2 * QB)];
  const int ca = (QA - 1) * pb.P + (QB - 1), cb = (QB - 1) * pb.P + (QA - 1);
  const int64_t na = st.counts[ca], nb = st.counts[cb];
  if (na + nb == 0) return;
  const int units = (int)gridDim.x / NXCD;
  const int ua = na == 0 ? 0 : (nb == 0 ? units : 1 + (int)((int64_t)(units - 2) * na / (na + nb)));
  const int unit = (int)blockIdx.x / NXCD;
  if (unit < ua)
    adj2d_class<FLUX, NV, QA, QB, 3>(pb, st, Slice(st.counts, st.list, ca, blockIdx.x, ua * NXCD, CPB), ubo, C, LMAX,
                                     xsm, g1s);
  else
    adj2d_class<FLUX, NV, QB, QA, 3>(pb, st,
                                     Slice(st.counts, st.list, cb, blockIdx.x - ua * NXCD, (units - ua) * NXCD, CPB),
                                     ubo, C, LMAX, xsm, g1s);
}

// Corners k whose node at offset j reads cell m along one direction of n
// cells: k = m - j (wrapped when periodic); with the transmissive clamp, an
// edge cell is also read by every corner whose node lies beyond it
// (k + j <= 0 for m = 0, k + j >= n - 1 for m = n - 1); corners run over
// [-1, n - 1] there.
__device__ __forceinline__ void corners_reading(int m, int j, int n, bool per, int& lo, int& hi) {
  lo = hi = m - j;
  if (per) return;
  if (m == 0) lo = -1;
  if (m == n - 1) hi = n - 1;
  lo = lo < -1 ? -1 : lo;
  hi = hi > n - 1 ? n - 1 : hi;
}

// 2D gather: cell m collects node (j1, j2) of every corner whose rectangle
// holds that node and whose node reads cell m (j2, corner row, j1, corner
// column: one fixed order).  P (the problem's largest half-width) is a
// template argument: with periodic boundaries every offset has exactly one
// corner, the loops unroll and the (2P)^2 class-map loads are issued
// together instead of one after another.
template <int NV, bool PER, int P>
__global__ __launch_bounds__(BLOCK) void k_gather2d(KProb pb, KStep st, const double* __restrict__ ubo,
                                                    const double* __restrict__ C, int LMAX, double* ubi) {
  const int64_t m = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  const int nx = (int)pb.nx, ny = (int)pb.ny, ioff = (int)pb.ioff;
  if (m >= (int64_t)nx * ny) return;
  constexpr bool per = PER;
  const int m1 = (int)(m % nx), m2 = (int)(m / nx);
  const int64_t plane = (int64_t)nx * ny;
  const int64_t nitems = pb.n1 * pb.n2;
  const int64_t cstride = nitems * LMAX;
  double acc[NV];
#pragma unroll
  for (int c = 0; c < NV; ++c) acc[c] = ubo[c * plane + m];
  if constexpr (PER) {
    int8_t cl[2 * P][2 * P];
    int64_t ek[2 * P][2 * P];
#pragma unroll
    for (int j2 = -P + 1; j2 <= P; ++j2)
#pragma unroll
      for (int j1 = -P + 1; j1 <= P; ++j1) {
        const int r2 = bc_index32(m2 - j2, ny, PERIODIC), r1 = bc_index32(m1 - j1, nx, PERIODIC);
        const int64_t e = (int64_t)r2 * pb.n1 + r1;
        ek[j2 + P - 1][j1 + P - 1] = e;
        cl[j2 + P - 1][j1 + P - 1] = st.cls[e];
      }
#pragma unroll
    for (int j2 = -P + 1; j2 <= P; ++j2)
#pragma unroll
      for (int j1 = -P + 1; j1 <= P; ++j1) {
        const int c0 = cl[j2 + P - 1][j1 + P - 1];
        if (c0 < 0) continue;
        const int q1 = c0 / P + 1, q2 = c0 % P + 1;
        if (j1 < -q1 + 1 || j1 > q1 || j2 < -q2 + 1 || j2 > q2) continue;
        const int64_t e = ek[j2 + P - 1][j1 + P - 1];
        const int64_t slot = (int64_t)(j2 + P - 1) * (2 * P) + (j1 + P - 1);
#pragma unroll
        for (int c = 0; c < NV; ++c) acc[c] += C[c * cstride + slot * nitems + e];
      }
#pragma unroll
    for (int c = 0; c < NV; ++c) ubi[c * plane + m] = acc[c];
    return;
  }
  for (int j2 = -P + 1; j2 <= P; ++j2) {
    int lo2, hi2;
    corners_reading(m2, j2, ny, per, lo2, hi2);
    for (int k2 = lo2; k2 <= hi2; ++k2) {
      const int r2 = per ? bc_index32(k2, ny, PERIODIC) : k2;
      for (int j1 = -P + 1; j1 <= P; ++j1) {
        int lo1, hi1;
        corners_reading(m1, j1, nx, per, lo1, hi1);
        for (int k1 = lo1; k1 <= hi1; ++k1) {
          const int r1 = per ? bc_index32(k1, nx, PERIODIC) : k1;
          const int64_t e = (int64_t)(r2 - ioff) * pb.n1 + (r1 - ioff);
          const int cl = st.cls[e];
          if (cl < 0) continue;
          const int q1 = cl / P + 1, q2 = cl % P + 1;
          if (j1 < -q1 + 1 || j1 > q1 || j2 < -q2 + 1 || j2 > q2) continue;
          const int64_t slot = (int64_t)(j2 + P - 1) * (2 * P) + (j1 + P - 1);
#pragma unroll
          for (int c = 0; c < NV; ++c) acc[c] += C[c * cstride + slot * nitems + e];
        }
      }
    }
  }
#pragma unroll
  for (int c = 0; c < NV; ++c) ubi[c * plane + m] = acc[c];
}

#define ACAT_CHECK_LAUNCH()                  \
  do {                                       \
    hipError_t e_ = hipGetLastError();       \
    if (e_ != hipSuccess) return e_;         \
  } while (0)

// The classes of a step of P <= 3 in launches whose blocks share the rounds of all
// their lists, taken in turn, the costliest class first: LOW, those of orders up to 2
// (two blocks per CU); EACH, all of P = 3 (one block); RECT2 and RECT3, the classes of
// highest order 2 and 3 without the square one, and with (1,1) for 2; REST, all of
// P = 3 without the square one (a scalar law's, two blocks).  Same arithmetic per
// corner as a launch per class.  Bound by FP64 issue at one or two waves per SIMD,
// and a launch per class ended each with most of the card idle: a class of a small
// grid has fewer rounds than the card has blocks.  A large grid's square class (P, P)
// keeps a launch of its own, in which it spills nothing and a scalar law's has twice
// the waves (adj_square_line).  Whole adjoint step, Euler, launches per class / these:
// 192^2 P = 3 276 us / 186, 512^2 P = 3 2547 / 2430, 600^2 P = 2 550 / 526 (without
// noise).  P = 4 keeps a launch per class: its rectangles of order 4 run in two
// launches each, and the body of all others beside them spills.
enum AdjClasses { LOW, EACH, RECT2, RECT3, REST };

template <int P, AdjClasses S>
struct AdjSet {
  struct Cls {
    int q1, q2, per_round, stride;
  };
  template <int Q1, int Q2>
  static constexpr Cls cls() {
    if (Q1 * Q2 == 1) return {1, 1, BLOCK, 0};
    return {Q1, Q2, Groups<4 * Q1 * Q2>::PER_BLOCK, adj_stride<4 * Q1 * Q2>()};
  }
  static constexpr Cls EVERY[9] = {cls<3, 3>(), cls<2, 3>(), cls<3, 2>(), cls<1, 3>(), cls<3, 1>(),
                                   cls<2, 2>(), cls<1, 2>(), cls<2, 1>(), cls<1, 1>()};   // costliest first
  static constexpr int FIRST = S == RECT2 ? 6 : S == RECT3 || S == REST ? 1 : S == EACH ? 0 : (P >= 2 ? 5 : 8);
  static constexpr int N = S == RECT3 ? 4 : 9 - FIRST;
  static constexpr Cls at(int k) { return EVERY[FIRST + k]; }
  static constexpr int max_stride() {
    int m = 1;
    for (int k = 0; k < N; ++k) m = at(k).stride > m ? at(k).stride : m;
    return m;
  }
  static constexpr int min_per_round() {
    int m = BLOCK;
    for (int k = 0; k < N; ++k) m = at(k).per_round < m ? at(k).per_round : m;
    return m;
  }
};

template <int FLUX, int NV, int P, AdjClasses S>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(S == LOW || S == RECT2 ? 2 : 1))) void k_adj2d_set(
    KProb pb, KStep st, const double* __restrict__ ubo, double* __restrict__ C, int LMAX) {
  using Set = AdjSet<P, S>;
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
      int cls[9], per_round[9];
    } t{};
    for (int k = 0; k < Set::N; ++k) {
      t.cls[k] = (Set::at(k).q1 - 1) * P + Set::at(k).q2 - 1;
      t.per_round[k] = Set::at(k).per_round;
    }
    return t;
  }();
  Chunks<Set::N, false> ck(st, tab, 0, blockIdx.x, gridDim.x, [&](int k, int& c, int& per_round) {
    c = sets.cls[k];
    per_round = sets.per_round[k];
  });
  auto run = [&](auto kc) {
    constexpr int k = decltype(kc)::value;
    if constexpr (k < Set::N) {
      constexpr auto c = Set::at(k);
      // computed at each chunk: kept for all classes at once it would spill
      int tid = threadIdx.x;
      double h = dt;
      asm volatile("" : "+v"(tid), "+v"(h));
      if constexpr (c.q1 == 1 && c.q2 == 1)
        adj2d_q11<FLUX, NV>(pb, st, tid, h, ck.items, ck.base, ck.end, ubo, C, LMAX);
      else
        adj2d_body<FLUX, NV, c.q1, c.q2, 3>(pb, st, tid, h, ck.items, ck.base, ck.end, ubo, C, LMAX, xsm,
                                            gxs + EdgeWeights::first(c.q1), gys + EdgeWeights::first(c.q2));
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

template <int FLUX, int NV, int P, AdjClasses S>
hipError_t launch_adjset(const KProb& pb, const KStep& st, const double* ubo, double* C, hipStream_t stream) {
  using Set = AdjSet<P, S>;
  static constexpr LaunchName name = class_launch_name<Set>("adjoint2d_");
  auto kern = k_adj2d_set<FLUX, NV, P, S>;
  static const int per_cu = [&] {
    int b = 0;
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, kern, BLOCK, 0) == hipSuccess && b > 0 ? b : 1;
  }();
  const int64_t rounds = pb.n1 * pb.n2 / Set::min_per_round() + NXCD * Set::N;
  const int grid = persistent_grid(kern, rounds * BLOCK, 0, BLOCK, per_cu);
  {
    ProfScope ps(name.s, stream);
    kern<<<grid, BLOCK, 0, stream>>>(pb, st, ubo, C, 4 * P * P);
  }
  ACAT_CHECK_LAUNCH();
  return hipSuccess;
}

// One order of a tile's interfaces: the wave's share of its rounds, the rounds of
// all orders dealt to the waves in turn.
template <int FLUX, int NV, int p>
__device__ __forceinline__ void adjtile_order(const KProb& pb, const KStep& st, double dt,
                                              const double* __restrict__ ubo, double* __restrict__ C, double* xs,
                                              const uint8_t* list, int k0, int first, int count, int& task) {
  using Adj = Adj1D<FLUX, NV, p>;
  constexpr int PER = Adj::Grp::PER_BLOCK;
  const int rounds = (count + PER - 1) / PER;
  if (task < rounds) {
    int lane = __lane_id();   // computed at each order: kept for all at once it would spill
    asm volatile("" : "+v"(lane), "+v"(dt));
    const Adj adj(lane);
    for (; task < rounds; task += NWAVE) {
      const int it = task * PER + adj.grp.g;
      const bool valid = adj.grp.in && it < count;
      const int32_t k = valid ? k0 + list[first + it] : 0;
      adj1d_body<FLUX, NV, p>(pb, st, adj, valid, k, dt, ubo, C, xs);
    }
  }
  task -= rounds;
}

template <int FLUX, int NV, int PM>
constexpr int adj_xs_doubles() {
  int m = Adj1D<FLUX, NV, 1>::LDS_DOUBLES;
  if constexpr (PM > 1) m = std::max(adj_xs_doubles<FLUX, NV, PM - 1>(), Adj1D<FLUX, NV, PM>::LDS_DOUBLES);
  return m;
}

template <int NV, int P>
constexpr int adj1d_waves() {
  return P <= 2 ? 3 : P == 3 || (NV == 1 && P <= 5) ? 2 : 1;
}

// The contributions of the interfaces of orders LO .. HI of a tile of T consecutive ones
// by one block, which groups them by order in LDS (mapped: by the class map, else by
// the recorded orders, which it writes to the map; counted: with the class counts).  Bound by FP64 issue at the one to
// three waves per SIMD that the Taylor history of the order leaves (spilled to reach
// one more it is slower: Burgers P = 6 2e5 cells 411 us in one, 541 in two); small
// problems by launches, of which lists and a kernel per order took six more.  Recorded
// step and adjoint, Euler, 30 % noise, by orders / by tiles: 20011 cells P = 3 (and a
// replayed step) 98 us / 53; 1e6 cells P = 3 627 / 516, P = 4 2274 / 1610, 4e5 cells P = 5
// 4418 / 2246, P = 6 20103 / 4795 (there the opaque history counts most); Burgers 1e6
// cells P = 5 824 / 595, P = 6 1306 / 1236, and nothing but order 1 129 / 117.
template <int FLUX, int NV, int P, int LO, int HI, bool TOP>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(adj1d_waves<NV, HI>()))) void k_adj1d(
    KProb pb, KStep st, int T, int mapped, int counted, const double* __restrict__ ubo, double* __restrict__ C) {
  if (LO > 1 && counted) {   // the step's class counts: nothing to do
    int any = 0;
    for (int p = LO; p <= HI; ++p) any |= st.counts[p - 1];
    if (any == 0) return;
  }
  __shared__ double xs[NWAVE][adj_xs_doubles<FLUX, NV, HI>()];
  __shared__ int wc[HI + 1][NWAVE];
  __shared__ uint8_t list[BLOCK];
  const int tid = threadIdx.x, lane = __lane_id(), wid = tid >> 6;
  const int32_t k0 = tile_item(blockIdx.x, T, 0, pb.nIx), k = tile_item(blockIdx.x, T, tid, pb.nIx);
  const double dt = step_dt(st);
  int ps = 0;
  if (k >= 0) {
    if (mapped) {
      ps = st.cls[k] + 1;
    } else {
      ps = st.ordx[k];
      if (ps < 1 || ps > P) {   // invalid recorded order: taken as 1, flagged
        ps = 1;
        atomicOr(st.status, 4u);
      }
      st.cls[k] = (int8_t)(ps - 1);
    }
  }
  unsigned long long mine = 0ull;
#pragma unroll
  for (int p = LO; p <= HI; ++p) {
    const unsigned long long b = __ballot(ps == p);
    if (ps == p) mine = b;
    if (lane == 0) wc[p][wid] = __popcll(b);
  }
  if constexpr (TOP) {
    const unsigned long long b = __ballot(ps == P);
    if (lane == 0) wc[0][wid] = __popcll(b);
  }
  __syncthreads();
  if (TOP && tid == 0) {
    int n = 0;
    for (int q = 0; q < NWAVE; ++q) n += wc[0][q];
    st.hist[blockIdx.x] = n;
  }
  int count[HI + 1], first[HI + 1], run = 0;
#pragma unroll
  for (int p = HI; p >= LO; --p) {
    first[p] = run;
    int pos = run;
    count[p] = 0;
#pragma unroll
    for (int q = 0; q < NWAVE; ++q) {
      const int n = __builtin_amdgcn_readfirstlane(wc[p][q]);
      if (q < wid) pos += n;
      count[p] += n;
    }
    if (ps == p) list[pos + __popcll(mine & ((1ull << lane) - 1ull))] = (uint8_t)tid;
    run += count[p];
  }
  __syncthreads();
  int task = __builtin_amdgcn_readfirstlane(wid);
  auto order = [&](auto pc) {
    constexpr int p = decltype(pc)::value;
    if constexpr (p >= LO && p <= HI)
      adjtile_order<FLUX, NV, p>(pb, st, dt, ubo, C, xs[wid], list, k0, first[p], count[p], task);
  };
  order(std::integral_constant<int, 6>{});
  order(std::integral_constant<int, 5>{});
  order(std::integral_constant<int, 4>{});
  order(std::integral_constant<int, 3>{});
  order(std::integral_constant<int, 2>{});
  order(std::integral_constant<int, 1>{});
}

// The interfaces of order P (by the class map) alone, in equal shares, one contiguous
// stretch of them per wave; counts: their number in each of ntiles tiles of T
// interfaces.  For the scalar laws' P = 6, at one wave per SIMD: of a tile's few
// rounds of order 6 the last left waves idle, and the last tiles the chip (1e6
// cells, 30 % noise, the orders from 3 on by tiles 1410 us, so 1236; advection 1135 and
// 1030).  Held to one wave the advection's round is 2 % faster, Burgers' 1 % slower.
template <int FLUX, int NV, int P>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(1, 1))) void k_adj1d_top(KProb pb, KStep st, const int32_t* counts, int ntiles, int T,
                                                     const double* __restrict__ ubo, double* __restrict__ C) {
  using Adj = Adj1D<FLUX, NV, P>;
  constexpr int PER = Adj::Grp::PER_BLOCK;
  __shared__ double xs[NWAVE][Adj::LDS_DOUBLES];
  __shared__ int32_t queue[NWAVE][64 + PER];
  __shared__ int wsum[NWAVE], tile0[NWAVE], skip0[NWAVE];
  const int tid = threadIdx.x, lane = __lane_id(), wid = wave_uniform(tid >> 6);
  // the prefix over the tiles, a stretch of them per thread, and in it each wave's first item
  const int per = (ntiles + BLOCK - 1) / BLOCK, t0 = min(tid * per, ntiles), t1 = min(t0 + per, ntiles);
  int mine = 0;
  for (int t = t0; t < t1; ++t) mine += counts[t];
  int before = mine;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int v = __shfl_up(before, off);
    if (lane >= off) before += v;
  }
  if (lane == 63) wsum[wid] = before;
  __syncthreads();
  before -= mine;
  int total = 0;
  for (int w = 0; w < NWAVE; ++w) {
    if (w < wid) before += wsum[w];
    total += wsum[w];
  }
  const int64_t waves = (int64_t)gridDim.x * NWAVE;
  const int64_t first = ((int64_t)(blockIdx.x % NXCD) * (gridDim.x / NXCD) + blockIdx.x / NXCD) * NWAVE;
  for (int w = 0; w < NWAVE; ++w) {
    int s = (int)((first + w) * total / waves) - before;
    if (s >= 0 && s < mine) {
      int t = t0;
      for (; s >= counts[t]; ++t) s -= counts[t];
      tile0[w] = t;
      skip0[w] = s;
    }
  }
  __syncthreads();
  int left = wave_uniform((int)((first + wid + 1) * total / waves - (first + wid) * total / waves));
  if (left == 0) return;
  int skip = wave_uniform(skip0[wid]);
  const Adj adj(lane);
  const double dt = step_dt(st);
  int32_t* q = queue[wid];
  int queued = 0;
  // 64 interfaces of a tile at a time, the next ones read ahead, tiles without any left out
  int t = wave_uniform(tile0[wid]), j = 0, window = t;
  auto filled = [&] { return __ballot(window + lane < ntiles && counts[window + lane] != 0); };
  auto has = [&](int t, int j) {
    const int64_t k = (int64_t)t * T + j + lane;
    return t < ntiles && j + lane < T && k < pb.nIx && st.cls[k] == P - 1;
  };
  unsigned long long some = filled();
  bool take = has(t, j);
  while (left > 0 && t < ntiles) {
    int tn = t, jn = j + 64;
    if (jn >= T) {
      jn = 0;
      for (++tn; tn < ntiles; tn = window + 64) {
        if (tn >= window + 64) {
          window = tn;
          some = filled();
        }
        const unsigned long long m = some >> (tn - window);
        if (m) {
          tn += __builtin_ctzll(m);
          break;
        }
      }
    }
    const bool next = has(tn, jn);
    const unsigned long long b = __ballot(take);
    const int rank = __popcll(b & ((1ull << lane) - 1ull)) - skip, n = __popcll(b);
    const int add = min(max(n - skip, 0), left);
    if (take && rank >= 0 && rank < add) q[queued + rank] = (int32_t)((int64_t)t * T + j + lane);
    skip = max(skip - n, 0);
    queued += add;
    left -= add;
    wave_sync();
    int done = 0;
    for (; queued - done >= PER || (left == 0 && done < queued); done += PER) {
      const bool valid = adj.grp.in && done + adj.grp.g < queued;
      adj1d_body<FLUX, NV, P>(pb, st, adj, valid, valid ? q[done + adj.grp.g] : 0, dt, ubo, C, xs[wid]);
    }
    if (left == 0) break;
    queued -= done;   // what is left, less than a round, to the front
    const int32_t rest = lane < queued ? q[done + lane] : 0;
    wave_sync();
    if (lane < queued) q[lane] = rest;
    t = tn;
    j = jn;
    take = next;
  }
}

// Interfaces up to which the adjoint takes all orders in one launch.  Above, the
// orders 1 and 2 have one of their own, at three waves per SIMD (a scalar law: eight),
// and the scalar laws' order 6 another; a launch more costs 3 to 5 us.  Recorded step
// and adjoint, one launch / split, without noise, with 30 %, and noise everywhere (all
// interfaces of order 1):
//   Euler P = 4    120000 cells 312 / 315, 249 / 253, 46 / 44; 200000 483 / 484, 397 / 396,
//                  62 / 52; 1e6 2305 / 2268, 1632 / 1604, 165 / 124
//   Euler P = 5    20000 206 / 207, 196 / 196, 31 / 33; 60000 544 / 536, 419 / 414, 48 / 42;
//                  200000 1602 / 1557, 1130 / 1101, 86 / 68
//   Euler P = 6    60000 819 / 805, 1103 / 1083, 48 / 46; 400000 3707 / 3620, 4896 / 4795, 112 / 87
//   Burgers P = 5  120000 132 / 132, 111 / 112, 44 / 43; 200000 202 / 202, 158 / 155, 52 / 51;
//                  1e6 811 / 797, 614 / 595, 122 / 106
//   Burgers P = 6  100000 264 / 278, 215 / 222, 46 / 42; 200000 492 / 477, 404 / 370, 64 / 58;
//                  1e6 1890 / 1670, 1411 / 1236, 171 / 117
// At P <= 3 and a scalar law's P = 4 the one kernel has two waves or more for all
// orders (Burgers P = 4 1e6 365 / 366, 289 / 290, 91 / 88).
template <int NV, int P>
constexpr int64_t adj1d_line() {
  return P < 4 || (NV == 1 && P == 4) ? INT64_MAX : NV == 1 ? 125000 : P == 4 ? 150000 : 50000;
}

// Tiles of the interfaces of orders LO .. HI, T interfaces each.  TOP: writes the number
// of those of order P > HI in each tile to st.hist.
template <int FLUX, int NV, int P, int LO, int HI, bool TOP = false>
hipError_t launch_adj1d(const KProb& pb, const KStep& st, bool mapped, bool counted, const double* ubo, double* C,
                        hipStream_t s, int* tile = nullptr) {
  auto kern = k_adj1d<FLUX, NV, P, LO, HI, TOP>;
  static const int per_cu = [&] {
    int b = 0;
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, kern, BLOCK, 0) == hipSuccess && b > 0 ? b : 1;
  }();
  const int T = tile_cells<HI>(pb.nIx, (int64_t)per_cu * num_cus(), 0, BLOCK);
  if (tile) *tile = T;
  static const char* const names[3] = {"adjoint1d", "adjoint1d_low", "adjoint1d_high"};
  ProfScope ps(names[LO == 1 && HI == P ? 0 : LO == 1 ? 1 : 2], s);
  kern<<<(unsigned)((pb.nIx + T - 1) / T), BLOCK, 0, s>>>(pb, st, T, mapped, counted, ubo, C);
  return hipGetLastError();
}

template <int FLUX, int NV, int P>
hipError_t adj1d_impl(const KProb& pb, const KStep& st, bool mapped, const double* ubo, double* ubi, double* C,
                      hipStream_t s) {
  hipError_t e;
  if (pb.nIx <= adj1d_line<NV, P>()) {
    if ((e = launch_adj1d<FLUX, NV, P, 1, P>(pb, st, mapped, mapped, ubo, C, s)) != hipSuccess) return e;
  } else if constexpr (P >= 4) {
    constexpr bool TOP = NV == 1 && P == 6;
    int T = 0;
    if ((e = launch_adj1d<FLUX, NV, P, 1, 2, TOP>(pb, st, mapped, mapped, ubo, C, s, &T)) != hipSuccess)
      return e;
    if ((e = launch_adj1d<FLUX, NV, P, 3, TOP ? P - 1 : P>(pb, st, true, mapped, ubo, C, s)) != hipSuccess) return e;
    if constexpr (TOP) {
      // the tiles' counts lie where a 2D step has its histograms, MAX_CLASSES for each 256 interfaces
      static_assert(NWAVE * Groups<4, 64>::PER_BLOCK * MAX_CLASSES >= 256, "the tiles' counts fit the histograms");
      auto kern = k_adj1d_top<FLUX, NV, P>;
      const int grid = persistent_grid(kern, pb.nIx, 0);
      ProfScope ps("adjoint1d_top", s);
      kern<<<grid, BLOCK, 0, s>>>(pb, st, st.hist, (int)((pb.nIx + T - 1) / T), T, ubo, C);
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
  }
  {
    ProfScope ps("gather1d", s);
    k_gather1d<NV, P><<<(unsigned)((pb.nx + BLOCK - 1) / BLOCK), BLOCK, 0, s>>>(pb, st, ubo, C, ubi);
  }
  ACAT_CHECK_LAUNCH();
  return hipSuccess;
}

template <int FLUX, int NV, int P, int Q1, int Q2>
hipError_t launch_adj2d(const KProb& pb, const KStep& st, const double* ubo, double* C, hipStream_t s) {
  if constexpr (Q1 <= P && Q2 <= P) {
    static const char* names[5][5] = {{"", "", "", "", ""},
                                      {"", "adjoint2d_q11", "adjoint2d_q12", "adjoint2d_q13", "adjoint2d_q14"},
                                      {"", "adjoint2d_q21", "adjoint2d_q22", "adjoint2d_q23", "adjoint2d_q24"},
                                      {"", "adjoint2d_q31", "adjoint2d_q32", "adjoint2d_q33", "adjoint2d_q34"},
                                      {"", "adjoint2d_q41", "adjoint2d_q42", "adjoint2d_q43", "adjoint2d_q44"}};
    // the rectangles with two recursions of orders 4 and 8 or 6 and 8 run
    // them in two launches (one recursion each, in order on the stream):
    // together in one kernel they exceed the register file several times
    constexpr bool SPLIT = Q1 != Q2 && Q1 >= 2 && Q2 >= 2 && Q1 + Q2 >= 6;
    if constexpr (Q1 == 1 && Q2 == 1) {
      // one lane per corner
      auto kern = k_adj2d_q11<FLUX, NV>;
      const int grid = persistent_grid(kern, pb.n1 * pb.n2, 0);
      ProfScope ps(names[1][1], s);
      kern<<<grid, BLOCK, 0, s>>>(pb, st, ubo, C, 4 * P * P);
    } else if constexpr (SPLIT) {
      auto k1 = k_adj2d<FLUX, NV, Q1, Q2, 1>;
      auto k2 = k_adj2d<FLUX, NV, Q1, Q2, 2>;
      ProfScope ps(names[Q1][Q2], s);
      k1<<<group_grid<(2 * Q1) * (2 * Q2)>(k1, pb.n1 * pb.n2, 0), BLOCK, 0, s>>>(pb, st, ubo, C, 4 * P * P);
      k2<<<group_grid<(2 * Q1) * (2 * Q2)>(k2, pb.n1 * pb.n2, 0), BLOCK, 0, s>>>(pb, st, ubo, C, 4 * P * P);
    } else {
      auto kern = k_adj2d<FLUX, NV, Q1, Q2>;
      const int grid = group_grid<(2 * Q1) * (2 * Q2)>(kern, pb.n1 * pb.n2, 0);
      ProfScope ps(names[Q1][Q2], s);
      kern<<<grid, BLOCK, 0, s>>>(pb, st, ubo, C, 4 * P * P);
    }
    ACAT_CHECK_LAUNCH();
  }
  return hipSuccess;
}

// The mirror classes (QA, QB) and (QB, QA), QA < QB, in one launch; only for
// the rectangles of orders up to 3 (those of order 4 keep one launch per class,
// the (1, 4) pair included: its device build gave wrong values).
template <int FLUX, int NV, int P, int QA, int QB>
hipError_t launch_adjpair2d(const KProb& pb, const KStep& st, const double* ubo, double* C, hipStream_t s) {
  static_assert(QA < QB && QB <= 3, "pairs of rectangles of orders up to 3 only");
  if constexpr (QB <= P) {
    static const char* names[4][4] = {{"", "", "", ""},
                                      {"", "", "adjoint2d_q12q21", "adjoint2d_q13q31"},
                                      {"", "", "", "adjoint2d_q23q32"},
                                      {"", "", "", ""}};
    auto kern = k_adj2d_pair<FLUX, NV, QA, QB>;
    // two runs of XCD groups: at least one per class
    const int grid = std::max(group_grid<(2 * QA) * (2 * QB)>(kern, pb.n1 * pb.n2, 0), 2 * NXCD);
    ProfScope ps(names[QA][QB], s);
    kern<<<grid, BLOCK, 0, s>>>(pb, st, ubo, C, 4 * P * P);
    ACAT_CHECK_LAUNCH();
  }
  return hipSuccess;
}

// Corners up to which the classes of P = 2 and 3 go in one launch; above, the square
// class (P, P) has its own, and the others one (Euler P = 3 two).  The line lies where
// the launch more is also small against a step in which next to nothing is smooth.
// Forward step and adjoint in us, one launch / split, without noise, with 30 % and
// 60 % of it, and noise everywhere:
//   Euler P = 2     350^2 200 / 197, 153 / 153, 111 / 114, 50 / 52; 512^2 408 / 384,
//                   306 / 291, 208 / 204, 78 / 80 (200 steps of a run with 84 % of the
//                   corners of class (1, 1): reverse pass 15.6 ms / 16.2); 600^2
//                   562 / 526, 418 / 400, 281 / 273, 94 / 95
//   Euler P = 3     350^2 1121 / 1101, 784 / 787, 479 / 487, 64 / 69
//   advection P = 2 300^2 76 / 76 without, 44 / 48 with noise everywhere; 350^2
//                   96 / 81, 80 / 72, 67 / 60, 48 / 47
//   advection P = 3 250^2 180 / 157, 142 / 126, 106 / 99, 49 / 57; 350^2 312 / 257,
//                   241 / 207, 167 / 150, 69 / 73
template <int NV, int P>
constexpr int64_t adj_square_line() {
  return NV == 1 ? (P == 3 ? 100000 : 120000) : P == 3 ? 150000 : 300000;
}

template <int FLUX, int NV, int P>
hipError_t adj2d_impl(const KProb& pb, const KStep& st, const double* ubo, double* ubi, double* C, hipStream_t s) {
  hipError_t e;
  if constexpr (P <= 3) {
    if (P == 1 || pb.n1 * pb.n2 <= adj_square_line<NV, P>()) {
      if ((e = launch_adjset<FLUX, NV, P, P == 3 ? EACH : LOW>(pb, st, ubo, C, s)) != hipSuccess) return e;
    } else if constexpr (P > 1) {
      if ((e = launch_adj2d<FLUX, NV, P, P, P>(pb, st, ubo, C, s)) != hipSuccess) return e;
      constexpr AdjClasses others = P == 2 ? RECT2 : NV == 1 ? REST : RECT3;
      if ((e = launch_adjset<FLUX, NV, P, others>(pb, st, ubo, C, s)) != hipSuccess) return e;
      if constexpr (others == RECT3)
        if ((e = launch_adjset<FLUX, NV, P, LOW>(pb, st, ubo, C, s)) != hipSuccess) return e;
    }
  } else {
    if ((e = launch_adj2d<FLUX, NV, P, 1, 1>(pb, st, ubo, C, s)) != hipSuccess) return e;
    if ((e = launch_adjpair2d<FLUX, NV, P, 1, 2>(pb, st, ubo, C, s)) != hipSuccess) return e;
    if ((e = launch_adj2d<FLUX, NV, P, 2, 2>(pb, st, ubo, C, s)) != hipSuccess) return e;
    if ((e = launch_adjpair2d<FLUX, NV, P, 1, 3>(pb, st, ubo, C, s)) != hipSuccess) return e;
    if ((e = launch_adjpair2d<FLUX, NV, P, 2, 3>(pb, st, ubo, C, s)) != hipSuccess) return e;
    if ((e = launch_adj2d<FLUX, NV, P, 3, 3>(pb, st, ubo, C, s)) != hipSuccess) return e;
    if ((e = launch_adj2d<FLUX, NV, P, 1, 4>(pb, st, ubo, C, s)) != hipSuccess) return e;
    if ((e = launch_adj2d<FLUX, NV, P, 4, 1>(pb, st, ubo, C, s)) != hipSuccess) return e;
    if ((e = launch_adj2d<FLUX, NV, P, 2, 4>(pb, st, ubo, C, s)) != hipSuccess) return e;
    if ((e = launch_adj2d<FLUX, NV, P, 4, 2>(pb, st, ubo, C, s)) != hipSuccess) return e;
    if ((e = launch_adj2d<FLUX, NV, P, 3, 4>(pb, st, ubo, C, s)) != hipSuccess) return e;
    if ((e = launch_adj2d<FLUX, NV, P, 4, 3>(pb, st, ubo, C, s)) != hipSuccess) return e;
    if ((e = launch_adj2d<FLUX, NV, P, 4, 4>(pb, st, ubo, C, s)) != hipSuccess) return e;
  }
  {
    ProfScope ps("gather2d", s);
    const unsigned gb = (unsigned)((pb.nx * pb.ny + BLOCK - 1) / BLOCK);
    if (pb.bc == PERIODIC) k_gather2d<NV, true, P><<<gb, BLOCK, 0, s>>>(pb, st, ubo, C, 4 * P * P, ubi);
    else k_gather2d<NV, false, P><<<gb, BLOCK, 0, s>>>(pb, st, ubo, C, 4 * P * P, ubi);
  }
  ACAT_CHECK_LAUNCH();
  return hipSuccess;
}

}  // namespace

hipError_t launch_adjoint(const KProb& pb, const KStep& st, bool mapped, const double* ubo, double* ubi, double* C,
                          hipStream_t s) {
  if (pb.dim == 1) {
    if (pb.flux == EUL) {
      switch (pb.P) {
        case 1: return adj1d_impl<EUL, 3, 1>(pb, st, mapped, ubo, ubi, C, s);
        case 2: return adj1d_impl<EUL, 3, 2>(pb, st, mapped, ubo, ubi, C, s);
        case 3: return adj1d_impl<EUL, 3, 3>(pb, st, mapped, ubo, ubi, C, s);
        case 4: return adj1d_impl<EUL, 3, 4>(pb, st, mapped, ubo, ubi, C, s);
        case 5: return adj1d_impl<EUL, 3, 5>(pb, st, mapped, ubo, ubi, C, s);
        case 6: return adj1d_impl<EUL, 3, 6>(pb, st, mapped, ubo, ubi, C, s);
      }
    } else if (pb.flux == BURG) {
      switch (pb.P) {
        case 1: return adj1d_impl<BURG, 1, 1>(pb, st, mapped, ubo, ubi, C, s);
        case 2: return adj1d_impl<BURG, 1, 2>(pb, st, mapped, ubo, ubi, C, s);
        case 3: return adj1d_impl<BURG, 1, 3>(pb, st, mapped, ubo, ubi, C, s);
        case 4: return adj1d_impl<BURG, 1, 4>(pb, st, mapped, ubo, ubi, C, s);
        case 5: return adj1d_impl<BURG, 1, 5>(pb, st, mapped, ubo, ubi, C, s);
        case 6: return adj1d_impl<BURG, 1, 6>(pb, st, mapped, ubo, ubi, C, s);
      }
    } else {
      switch (pb.P) {
        case 1: return adj1d_impl<ADV, 1, 1>(pb, st, mapped, ubo, ubi, C, s);
        case 2: return adj1d_impl<ADV, 1, 2>(pb, st, mapped, ubo, ubi, C, s);
        case 3: return adj1d_impl<ADV, 1, 3>(pb, st, mapped, ubo, ubi, C, s);
        case 4: return adj1d_impl<ADV, 1, 4>(pb, st, mapped, ubo, ubi, C, s);
        case 5: return adj1d_impl<ADV, 1, 5>(pb, st, mapped, ubo, ubi, C, s);
        case 6: return adj1d_impl<ADV, 1, 6>(pb, st, mapped, ubo, ubi, C, s);
      }
    }
  } else {
    if (pb.flux == EUL) {
      switch (pb.P) {
        case 1: return adj2d_impl<EUL, 4, 1>(pb, st, ubo, ubi, C, s);
        case 2: return adj2d_impl<EUL, 4, 2>(pb, st, ubo, ubi, C, s);
        case 3: return adj2d_impl<EUL, 4, 3>(pb, st, ubo, ubi, C, s);
        case 4: return adj2d_impl<EUL, 4, 4>(pb, st, ubo, ubi, C, s);
      }
    } else {
      switch (pb.P) {
        case 1: return adj2d_impl<ADV, 1, 1>(pb, st, ubo, ubi, C, s);
        case 2: return adj2d_impl<ADV, 1, 2>(pb, st, ubo, ubi, C, s);
        case 3: return adj2d_impl<ADV, 1, 3>(pb, st, ubo, ubi, C, s);
        case 4: return adj2d_impl<ADV, 1, 4>(pb, st, ubo, ubi, C, s);
      }
    }
  }
  return hipErrorInvalidValue;
}

}  // namespace acat
