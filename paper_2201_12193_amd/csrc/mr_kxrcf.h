/* What the two KXRCF kernels of the 2D equations share (mr_kxrcf2d.hip,
 * mr_kxrcf2w.hip): the strip and its characteristic-wise face data. */
#pragma once
#include "mr_common.h"

#define KX_W 64                       /* reconstructed columns of a strip */
#define KX_XW (KX_W + 2)              /* staged columns                   */

/* face data of one direction D of the characteristic-wise Step 1 (2D
   Euler, four components staged; see mr_char2): each field projected from
   the stencil, reconstructed, and mapped back at the points the indicator
   reads -- the density at all sixteen points (its norm), the density and
   the normal momentum at the points of the two faces normal to D.
   f[0..1] / f[4..5] (D = 0: left, right) or f[2..3] / f[6..7] (D = 1:
   bottom, top), means and velocities; *nrm is raised to max |rho|.  order()
   keeps the compiler from moving loads over it: the constant table stays in
   LDS, not in registers over the loop of the fields. */
template <bool BP, int D, class Order>
MR_INL void kx_face_data_ch(const double (*mom)[12 * KX_XW], int s0, int s1, int s2, int col,
                            const mr_wconst& W, double gam, double f[9], double* nrm, Order order) {
  double u0[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) u0[c] = mom[s1][(3 * c + 0) * KX_XW + col];
  const mr_char2 e = mr_char2_state<D>(u0, gam);
  double rho[16], mn[8];
#pragma unroll
  for (int q = 0; q < 16; ++q) rho[q] = 0.0;
#pragma unroll
  for (int q = 0; q < 8; ++q) mn[q] = 0.0;
#pragma unroll 1
  for (int k = 0; k < 4; ++k) {
    order();
    double lk[4];
    mr_char2_left<D>(e, k, lk);
    double u[9], v[9], w[9], q[16];
#pragma unroll
    for (int l = 0; l < 9; ++l) {
      const int dx = l % 3 - 1, slot = l < 3 ? s0 : (l < 6 ? s1 : s2);
      u[l] = v[l] = w[l] = 0.0;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        u[l] += lk[c] * mom[slot][(3 * c + 0) * KX_XW + col + dx];
        v[l] += lk[c] * mom[slot][(3 * c + 1) * KX_XW + col + dx];
        w[l] += lk[c] * mom[slot][(3 * c + 2) * KX_XW + col + dx];
      }
    }
    mr_recon2d<BP>(u, v, w, W, q);
    /* column k of R: density entry 1, 1, 0, 1; normal momentum vn - c, vn, 0, vn + c */
    const double rr = k == 2 ? 0.0 : 1.0;
    const double rn = k == 0 ? e.vn - e.c : (k == 1 ? e.vn : (k == 2 ? 0.0 : e.vn + e.c));
#pragma unroll
    for (int p = 0; p < 16; ++p) rho[p] += rr * q[p];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const int pa = D == 0 ? 4 * m : m, pb = D == 0 ? 3 + 4 * m : 12 + m;
      mn[m] += rn * q[pa];
      mn[4 + m] += rn * q[pb];
    }
  }
#pragma unroll
  for (int p = 0; p < 16; ++p) *nrm = fmax(*nrm, fabs(rho[p]));
  double sa = 0.0, sb = 0.0, va = 0.0, vb = 0.0;
  double ia[4], ib[4];
  if (D == 0) { mr_recip4(rho[0], rho[4], rho[8], rho[12], ia); mr_recip4(rho[3], rho[7], rho[11], rho[15], ib); }
  else { mr_recip4(rho[0], rho[1], rho[2], rho[3], ia); mr_recip4(rho[12], rho[13], rho[14], rho[15], ib); }
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    const int pa = D == 0 ? 4 * m : m, pb = D == 0 ? 3 + 4 * m : 12 + m;
    sa += glw(m) * rho[pa];
    sb += glw(m) * rho[pb];
    va += glw(m) * (mn[m] * ia[m]);
    vb += glw(m) * (mn[4 + m] * ib[m]);
  }
  f[2 * D] = sa; f[2 * D + 1] = sb;
  f[4 + 2 * D] = va; f[5 + 2 * D] = vb;
}
