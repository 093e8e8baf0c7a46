// One wave of 1D interfaces: the CAT2p recursion (Sec. 2.2) with one lane per
// stencil node, and the FL-CAT2 blend (Sec. 3.1).  Shared by the per-class
// kernels, the tile kernels and the batched step, so that all of them round
// alike: every weighted sum of the recursion is a chain of fused
// multiply-adds in index order, nothing else is contracted (the library is
// built with -ffp-contract=off).
#pragma once

#include <hip/hip_runtime.h>

#include "step_common.hpp"

namespace acat {
namespace {

// BS threads share `xs` (LDS_DOUBLES doubles).  The groups of every 1D order
// are packed per wavefront, so the exchange is ordered by the wave's own
// in-order LDS operations: one buffer serves all levels.
template <int FLUX, int NV, int p, int BS>
struct Cat1D {
  static constexpr int L = 2 * p;               // lanes per interface = stencil nodes
  using Grp = Groups<L, BS>;
  static_assert(Grp::WAVE_LOCAL, "1D groups never span two waves");
  static constexpr int PER_ROUND = Grp::PER_BLOCK;
  static constexpr int SL = L + 1;              // LDS slots per interface (one pad slot against bank conflicts)
  static constexpr int NS = Grp::TOTAL * SL;    // slots per component, idle lanes included
  static constexpr int LDS_DOUBLES = NV * NS;

  int g, a;        // interface of the round, node of its stencil (offset a - p + 1)
  bool in;         // false for idle lanes
  double g1[L];    // first-derivative weights at this node

  __device__ __forceinline__ explicit Cat1D(int tid) {
    const Grp grp(tid);
    g = grp.g;
    a = grp.node;
    in = grp.in;
#pragma unroll
    for (int l = 0; l < L; ++l) g1[l] = TB.G1[p][a][l];
  }

  // CAT2p flux from this lane's node state u: component a on the lanes a < NV
  // (F0), component a + L too where NV > L (F1).
  __device__ __forceinline__ void flux(const Phys& ph, const double (&u)[NV], double lam, double* xs, double& F0,
                                       double& F1) const {
    const int gb = g * SL, slot = gb + a;
    double fh0[NV], cur[NV], S[NV];
    flux1d<FLUX, NV>(ph, u, fh0);
    // S = sum_k Fh^{k-1} / k! at this node (the CAT flux, summed node by node)
#pragma unroll
    for (int c = 0; c < NV; ++c) {
      cur[c] = fh0[c];
      S[c] = fma(TB.INVFACT[1], fh0[c], 0.0);
    }
    // Taylor predictions W_r = u + sum_{l<kk} r^l/l! U^l, U^l = dt^l u~^(l), at the
    // time nodes r != 0, one term added per level (same fma chain as summing from u)
    double W[L][NV];
#pragma unroll
    for (int ri = 0; ri < L; ++ri)
#pragma unroll
      for (int c = 0; c < NV; ++c) W[ri][c] = u[c];
#pragma unroll
    for (int kk = 2; kk <= 2 * p; ++kk) {
      // share Fh^{kk-2} of every node of the stencil
#pragma unroll
      for (int c = 0; c < NV; ++c) xs[c * NS + slot] = cur[c];
      Grp::sync();
      // U^{kk-1} = -lambda * (spatial derivative of Fh^{kk-2} at this node)
      double Uk[NV];
#pragma unroll
      for (int c = 0; c < NV; ++c) {
        double sacc = 0.0;
#pragma unroll
        for (int l = 0; l < L; ++l) sacc = fma(g1[l], xs[c * NS + gb + l], sacc);
        Uk[c] = -lam * sacc;
      }
      Grp::sync();
#pragma unroll
      for (int ri = 0; ri < L; ++ri) {
        const int r = ri - p + 1;
        if (r == 0) continue;
#pragma unroll
        for (int c = 0; c < NV; ++c) W[ri][c] = fma(TB.TAYLOR[r + PMAX - 1][kk - 1], Uk[c], W[ri][c]);
      }
      // flux at the Taylor-predicted states of the time nodes r, and its
      // (kk-1)-th time derivative at r = 0
      double nxt[NV];
#pragma unroll
      for (int c = 0; c < NV; ++c) nxt[c] = 0.0;
#pragma unroll
      for (int ri = 0; ri < L; ++ri) {
        const int r = ri - p + 1;
        // a time node whose weight is exactly zero adds nothing: its flux
        // is not evaluated (the same sum for finite values)
        if (TB.GT[p][kk - 1][ri] == 0.0) continue;
        double fr[NV];
        if (r == 0) {
#pragma unroll
          for (int c = 0; c < NV; ++c) fr[c] = fh0[c];
        } else {
          flux1d<FLUX, NV>(ph, W[ri], fr);
        }
#pragma unroll
        for (int c = 0; c < NV; ++c) nxt[c] = fma(TB.GT[p][kk - 1][ri], fr[c], nxt[c]);
      }
#pragma unroll
      for (int c = 0; c < NV; ++c) {
        cur[c] = nxt[c];
        S[c] = fma(TB.INVFACT[kk], nxt[c], S[c]);
      }
    }
    // F_c = sum_j eta_j S_j,c
#pragma unroll
    for (int c = 0; c < NV; ++c) xs[c * NS + slot] = S[c];
    Grp::sync();
    F0 = 0.0;
    F1 = 0.0;
    if (a < NV) {
#pragma unroll
      for (int l = 0; l < L; ++l) F0 = fma(TB.ETA[p][l], xs[a * NS + gb + l], F0);
      if (NV > L && a + L < NV) {
#pragma unroll
        for (int l = 0; l < L; ++l) F1 = fma(TB.ETA[p][l], xs[((a + L) % NV) * NS + gb + l], F1);
      }
    }
    Grp::sync();
  }
};

// Superbee weight psi^1 and Rusanov speed of an interface that takes order 1;
// v holds its window, offsets -G+1 .. G.
template <int FLUX, int NV, int G>
__device__ __forceinline__ void low_order_weights(const Phys& ph, int flags, const double (&v)[NV][2 * G],
                                                  double& psi1, double& al) {
  psi1 = limiter<NV, G>(v);
  if constexpr (NV == 1) {
    if (flags & FLAG_PSI1_ROE) psi1 = limiter_roe<FLUX, G>(ph, v, 0);
  }
  double uL[NV], uR[NV];
#pragma unroll
  for (int c = 0; c < NV; ++c) {
    uL[c] = v[c][G - 1];
    uR[c] = v[c][G];
  }
  al = fmax(spectral_radius<FLUX, 1, NV>(ph, uL, 0), spectral_radius<FLUX, 1, NV>(ph, uR, 0));
}

// FL-CAT2 (Sec. 3.1), component c: psi^1 CAT2 + (1 - psi^1) F^lo between the
// states uL and uR of the interface's two cells.
template <int FLUX, int NV>
__device__ __forceinline__ double fl_cat2(const Phys& ph, int flags, const double (&uL)[NV], const double (&uR)[NV],
                                          int c, double F, double psi, double al, double alf) {
  double fL[NV], fR[NV];
  flux1d<FLUX, NV>(ph, uL, fL);
  flux1d<FLUX, NV>(ph, uR, fR);
  double ul = 0.0, ur = 0.0, fl = 0.0, fr = 0.0;
#pragma unroll
  for (int cc = 0; cc < NV; ++cc)
    if (cc == c) {
      ul = uL[cc];
      ur = uR[cc];
      fl = fL[cc];
      fr = fR[cc];
    }
  const double flo = lo_flux<FLUX, 1, NV>(ph, flags, 0, uL, uR, fl, fr, ul, ur, al, alf);
  return psi * F + (1.0 - psi) * flo;
}

}  // namespace
}  // namespace acat
