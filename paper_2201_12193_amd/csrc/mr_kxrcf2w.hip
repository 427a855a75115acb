/* The 2D KXRCF indicator kernel of small launches (its own translation unit:
 * it keeps the constant table of the reconstruction in LDS, see
 * mr_device.h). */
#define MR_KT_IN_LDS 1
#include "mr_kxrcf.h"

/* =============================== 2D Euler KXRCF (tc = 1), one wave a strip */
/* The flags of k2_kxrcf for launches whose strips do not fill the GPU, where
 * a launch lasts as long as one strip: a wave (one per work group) owns a
 * strip of 62 flag columns and sweeps it upward row by row, one lane per
 * cell of the strip plus one ring column each side; Step 1 is that of the
 * unmodified stage input.  The moments of four rows (the planes the
 * indicator reads, two more columns) sit in an LDS ring, each loaded from
 * HBM once per strip with the boundary condition applied when it is stored,
 * a row ahead of its use.  No other wave is involved, so there is no
 * barrier in the sweep, and a strip may be as low as one row (the four
 * waves of k2_kxrcf take four rows a step and two barriers): the neighbours
 * in x are lanes, and the row below waits in registers (its face data and
 * the sums of eq. (KXRCF_) so far) until its top face is decided.
 *
 * The velocities enter the test by the sign of their face average only.
 * The value of a momentum at a face point is a convex combination of the
 * p_l, so it differs from the cell average u_5 by at most
 * a sum of the stencil's |u_j - u_5| and |first moments| with fixed factors
 * (kx_bound): where |u_5| exceeds that (and the density is
 * positive at the face points) the velocity has u_5's sign at all of them.
 * Rows whose 64 cells all agree need no Step 1 of that momentum: 35
 * operations decide instead of 450.  In x the row decides for itself; in y
 * a face between two rows of the same sign is decided, any other face takes
 * the velocities of both rows (the lower row's Step 1 again if it had been
 * left out).  The decision is the one the velocities give, so the flags are
 * the same; a NaN fails every comparison and takes the full path.
 *
 * A launch has a wave a SIMD at most, which may hold all its registers.
 * What bounds it: the chain of a lone wave, 11.5 us and 5.3 us a row where
 * every velocity is formed; strips are one to three rows high therefore.
 * Against k2_kxrcf: component-wise 22.4 -> 15.9 us at 96^2, 24 -> 23 at 331
 * x 257, 33 -> 29 at 400^2, characteristic-wise 72 -> 61 us at 96^2.
 * Launches that give the GPU more strips stay with k2_kxrcf (512^2: 33
 * against 39 us, characteristic-wise 159 against 255; with the sides' data
 * of an 800 x 200 double Mach reflection 43 against 65).  Far above that the
 * shortcut for the velocities would make this kernel the faster one again
 * (98 -> 89 us at 1024^2), but the learned indicator is an alternative there
 * that is to cost less than the KXRCF test. */
#define KX_MR 4                       /* moment ring rows                 */

/* the wave's LDS writes are ordered before its later reads (the LDS takes a
   wave's accesses in order; the compiler must not move them).  A fence, not
   an asm statement: with the latter ahead of them the loads of the instance
   descriptor are no longer scalar loads, and the kernel waits for them in
   every row */
MR_INL void kx_order() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }
/* value of the lane before / after in the wave (0 beyond the ends) */
template <int CTRL>
MR_INL double kx_lane(double v) {
  const long long b = __builtin_bit_cast(long long, v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffll), CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xF, 0xF, true);
  return __builtin_bit_cast(double, ((long long)hi << 32) | (long long)(unsigned)lo);
}
MR_INL double kx_left(double v) { return kx_lane<0x138>(v); }    /* wave_shr:1 */
MR_INL double kx_right(double v) { return kx_lane<0x130>(v); }   /* wave_shl:1 */

/* stencil of component c of the cell at staged column col, rows in slots s0, s1, s2 */
template <int NPL>
MR_INL void kx_stencil(const double (*mom)[NPL * KX_XW], int s0, int s1, int s2, int col, int c, double u[9],
                       double v[9], double w[9]) {
#pragma unroll
  for (int l = 0; l < 9; ++l) {
    const int dx = l % 3 - 1, slot = l < 3 ? s0 : (l < 6 ? s1 : s2);
    u[l] = mom[slot][(3 * c + 0) * KX_XW + col + dx];
    v[l] = mom[slot][(3 * c + 1) * KX_XW + col + dx];
    w[l] = mom[slot][(3 * c + 2) * KX_XW + col + dx];
  }
}

/* how far a value of Step 1 at a face point may be from the cell average
   (see the head of this file): with the nonlinear weights in [0, 1] and
   adding to 1 it lies among the p_l = S_l/gbar_l q_l - S_{l-1}/gbar_l q_{l-1};
   entry g multiplies the magnitudes of the data of group g */
struct kx_bound {
  double ue, uc, m0, me, mc;
};
MR_INL kx_bound kx_bounds(const mr_wconst& W) {
#define KX_B(G)                                                                        \
  fmax(W.sg[1] * MR_BND_Q2_##G, fmax(W.sg[2] * MR_BND_Q3_##G + W.sgn[1] * MR_BND_Q2_##G, \
                                     W.sg[3] * MR_BND_Q4_##G + W.sgn[2] * MR_BND_Q3_##G))
  return kx_bound{KX_B(UE), KX_B(UC), KX_B(M0), KX_B(ME), KX_B(MC)};
#undef KX_B
}
/* sign of component c at every face point of the cell: 1 or -1, or 0 where
   the bound leaves it open (1 % of the average covers the rounding; moments
   beyond 1e30, where the weights' products may overflow, are left open, and
   a NaN anywhere in the stencil spreads through the sum) */
template <int NPL>
MR_INL int kx_sign(const double (*mom)[NPL * KX_XW], int s0, int s1, int s2, int col, int c, const kx_bound& B) {
  double u[9], v[9], w[9];
  kx_stencil<NPL>(mom, s0, s1, s2, col, c, u, v, w);
  double b = B.m0 * fabs(v[4]), d = B.m0 * fabs(w[4]);
#pragma unroll
  for (int l = 0; l < 9; ++l) {
    const bool corner = l % 2 == 0;
    if (l != 4) b = fma(corner ? B.uc : B.ue, fabs(u[l] - u[4]), b);
    /* the maps read the x moments of the columns beside and the cell's own,
       the y moments of the rows below and above and the cell's own */
    if (l % 3 != 1) d = fma(corner ? B.mc : B.me, fabs(v[l]), d);
    if (l / 3 != 1) d = fma(corner ? B.mc : B.me, fabs(w[l]), d);
  }
  const double a = fabs(u[4]);
  if (!(0.99 * a > b + d) || !(a < 1e30)) return 0;
  return u[4] > 0.0 ? 1 : -1;
}

/* the sign all lanes of the wave agree on, or 0 */
MR_INL int kx_agree(int s) {
  if (__ballot(s > 0) == ~0ull) return 1;
  if (__ballot(s < 0) == ~0ull) return -1;
  return 0;
}

/* NK: components the indicator reads (3: rho and the momenta; 4 with the
   characteristic-wise Step 1, whose fields mix all components).  Work item:
   flag columns x0 .. x0+61, flag rows y0 .. y0+rows-1 of the extended flag
   range [-2, n+2)^2 (y0 >= -2).  No per-side boundary data. */
template <int NK, bool BP>
__global__ __launch_bounds__(KX_W) __attribute__((amdgpu_waves_per_eu(1))) void k2_kxrcf_few(const mr_inst* __restrict__ insts, const mr_tile2* __restrict__ tiles, int ntiles, int stage) {
  mr_kt_fill();
  constexpr int NPL = 3 * NK;
  __shared__ double mom[KX_MR][NPL * KX_XW];              /* [row][plane][column] */
  const int cx = threadIdx.x, col = cx + 1;
  for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
    const mr_tile2 tl = tiles[t];
    const mr_inst& I = insts[tl.inst];
    if (stage < 3 && !I.active) continue;
    const MR_GLB double* U = mr_gp(stage < 3 ? I.p_in[stage] : I.buf[0]);
    MR_GLB unsigned char* fl = mr_gp(I.flags[(stage == 0 || stage == 3) ? 0 : 1]);
    MR_GLB double* aleph = mr_gp(I.aleph);
    const long long P = I.plane;
    const int nx = I.nx;
    const int xs = tl.x0 - 2, x = xs + col;      /* staged column 0; this lane's cell */
    const int ylast = tl.y0 + tl.rows;           /* last reconstructed row */
    const kx_bound B = kx_bounds(I.W);
    /* staging: the lane's column of every plane, and one element of the last
       two columns for the first 2 NPL lanes */
    const bool ext = cx < 2 * NPL;
    const int ep = ext ? cx >> 1 : 0, ec = KX_W + (cx & 1);
    int kx = 0, kxe = 0;
    const int ii = mr_fold(xs + cx, nx, I.bcx, &kx), iie = mr_fold(xs + ec, nx, I.bcx, &kxe);
    const bool xplain = (xs >= 0 || (I.bcx & 3) == 0) && (xs + KX_XW <= nx || ((I.bcx >> 2) & 3) == 0);
    const MR_GLB double* ue = U + (long long)ep * P + iie;
    auto slot = [&](int y) { return (y - tl.y0 + 2) & (KX_MR - 1); };   /* y >= y0 - 2 */
    auto fetch = [&](int y, double* pf, double* pe, int* ky) {
      const long long jj = (long long)mr_fold(y, I.ny, I.bcy, ky) * nx;   /* uniform */
#pragma unroll
      for (int q = 0; q < NPL; ++q) pf[q] = (U + q * P + jj)[ii];
      if (ext) *pe = ue[jj];
    };
    auto ghost = [&](double v, int pl, int kxx, int ky) {
      const int c = pl / 3, m = pl % 3;
      const bool neg = (kxx == 2 && mr_refl_flip(c, m, 0)) != (ky == 2 && mr_refl_flip(c, m, 1));
      return (m != 0 && (kxx == 1 || ky == 1)) ? 0.0 : (neg ? -v : v);
    };
    auto store = [&](int y, const double* pf, double pe, int ky) {
      kx_order();
      double* d = mom[slot(y)];
      if (xplain && ky == 0) {
#pragma unroll
        for (int q = 0; q < NPL; ++q) d[q * KX_XW + cx] = pf[q];
        if (ext) d[ep * KX_XW + ec] = pe;
      } else {
#pragma unroll
        for (int q = 0; q < NPL; ++q) d[q * KX_XW + cx] = ghost(pf[q], q, kx, ky);
        if (ext) d[ep * KX_XW + ec] = ghost(pe, ep, kxe, ky);
      }
      kx_order();
    };
    /* prologue: moment rows y0-2 .. y0, their loads in flight together */
    {
      double pf[3][NPL], pe[3] = {0.0, 0.0, 0.0};
      int ky[3] = {0, 0, 0};
#pragma unroll
      for (int k = 0; k < 3; ++k) fetch(tl.y0 - 2 + k, pf[k], &pe[k], &ky[k]);
#pragma unroll
      for (int k = 0; k < 3; ++k) store(tl.y0 - 2 + k, pf[k], pe[k], ky[k]);
    }
    /* nothing in flight on entry: the waits of the sweep would otherwise
       cover these loads in every row, and with them the row's flag stores */
    __builtin_amdgcn_s_waitcnt(0x0F70);   /* vmcnt(0) */
    /* the row below: its sums so far, density norm, top face average, the
       density at its top points, the velocity of its top face (if act) */
    double J0 = 0.0, len0 = 0.0, nrm0 = 0.0, st0 = 0.0, vt0 = 0.0, rt0[4] = {1.0, 1.0, 1.0, 1.0};
    int sy0 = 0;          /* its agreed sign in y, 0 none     */
    bool act0 = false;    /* vt0 holds the velocity (uniform) */
#pragma unroll 1
    for (int r = tl.y0 - 1; r <= ylast; ++r) {
      /* moment row r+2 for the next step (rows past ylast+1 are not read) */
      double pf[NPL], pe = 0.0;
      int ky = 0;
      fetch(r + 2, pf, &pe, &ky);
      const int s0 = slot(r - 1), s1 = slot(r), s2 = slot(r + 1), sm = slot(r + 2) /* = slot(r - 2) */;
      double sl = 0.0, sr = 0.0, sb = 0.0, st = 0.0, nrm = 0.0;
      double vl = 0.0, vr = 0.0, vb = 0.0, vt = 0.0;
      double rt[4] = {1.0, 1.0, 1.0, 1.0};
      int sx = 0, sy = 0;
      bool act = true;
      if constexpr (NK == 4) {
        /* characteristic-wise Step 1: x faces from the x set, y faces from the y set */
        double f[9];
        f[8] = 0.0;
        kx_face_data_ch<BP, 0>(mom, s0, s1, s2, col, I.W, I.gam, f, &f[8], [] { kx_order(); });
        kx_face_data_ch<BP, 1>(mom, s0, s1, s2, col, I.W, I.gam, f, &f[8], [] { kx_order(); });
        sl = f[0]; sr = f[1]; sb = f[2]; st = f[3];
        vl = f[4]; vr = f[5]; vb = f[6]; vt = f[7];
        nrm = f[8];
      } else {
        double u[9], v[9], w[9], q[16];
        kx_stencil<NPL>(mom, s0, s1, s2, col, 0, u, v, w);
        mr_recon2d<BP>(u, v, w, I.W, q);
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          sl += glw(m) * q[0 + 4 * m];
          sr += glw(m) * q[3 + 4 * m];
          sb += glw(m) * q[m];
          st += glw(m) * q[12 + m];
        }
#pragma unroll
        for (int k = 0; k < 16; ++k) nrm = fmax(nrm, fabs(q[k]));
        {
          /* density positive (and moderate) at the face points? */
          double lo = q[0];
#pragma unroll
          for (int k = 1; k < 16; ++k)
            if (k % 4 == 0 || k % 4 == 3 || k < 4 || k >= 12) lo = fmin(lo, q[k]);
          const bool pos = lo > 1e-30 && nrm < 1e30;   /* (a NaN coefficient reaches every point) */
#pragma unroll
          for (int m = 0; m < 4; ++m) rt[m] = q[12 + m];
          kx_order();
          sx = kx_agree(pos ? kx_sign<NPL>(mom, s0, s1, s2, col, 1, B) : 0);
          kx_order();
          sy = kx_agree(pos ? kx_sign<NPL>(mom, s0, s1, s2, col, 2, B) : 0);
          kx_order();
          if (sx == 0 && r >= tl.y0 && r < ylast) {   /* the x velocities of the row's flags */
            double irl[4], irr[4], m[16];
            mr_recip4(q[0], q[4], q[8], q[12], irl);
            mr_recip4(q[3], q[7], q[11], q[15], irr);
            kx_stencil<NPL>(mom, s0, s1, s2, col, 1, u, v, w);
            mr_recon2d<BP>(u, v, w, I.W, m);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              vl += glw(k) * (m[0 + 4 * k] * irl[k]);
              vr += glw(k) * (m[3 + 4 * k] * irr[k]);
            }
          }
          act = false;
          if (r >= tl.y0 && !(sy != 0 && sy == sy0)) {
            /* the face to the row below is open: both rows' velocities (the
               lower row's Step 1 if it was left out, its rows r-2 .. r) */
            kx_order();
            double ir[4], m[16];
            if (!act0) {
              mr_recip4(rt0[0], rt0[1], rt0[2], rt0[3], ir);
              kx_stencil<NPL>(mom, sm, s0, s1, col, 2, u, v, w);
              mr_recon2d<BP>(u, v, w, I.W, m);
              vt0 = 0.0;
#pragma unroll
              for (int k = 0; k < 4; ++k) vt0 += glw(k) * (m[12 + k] * ir[k]);
              kx_order();
            }
            double it[4];
            mr_recip4(q[0], q[1], q[2], q[3], ir);
            mr_recip4(q[12], q[13], q[14], q[15], it);
            kx_stencil<NPL>(mom, s0, s1, s2, col, 2, u, v, w);
            mr_recon2d<BP>(u, v, w, I.W, m);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              vb += glw(k) * (m[k] * ir[k]);
              vt += glw(k) * (m[12 + k] * it[k]);
            }
            act = true;
          }
        }
      }
      /* the slot of row r-2 is free; ahead of the flags, so that the wait for
         the fetched row does not cover their stores */
      if (r + 2 <= ylast + 1) store(r + 2, pf, pe, ky);
      {
#pragma clang fp contract(off)
        double J = 0.0, len = 0.0;
        if (r >= tl.y0 && r < ylast) {
          /* x faces: the neighbours' values from the lanes beside */
          const double srl = kx_left(sr), slr = kx_right(sl);
          double fvl, fvr;
          if (NK == 3 && sx != 0) {
            fvl = fvr = (double)sx;
          } else {
            fvl = 0.5 * (vl + kx_left(vr));
            fvr = 0.5 * (vr + kx_right(vl));
          }
          if (fvl > 0.0 && !mr_wall(x, nx, I.bcx)) { J += I.dy * (sl - srl); len += I.dy; }
          if (-fvr > 0.0 && !mr_wall(x + 1, nx, I.bcx)) { J += I.dy * (sr - slr); len += I.dy; }
        }
        if (r >= tl.y0) {
          /* the face between the row below and this one */
          const double v = (NK == 3 && sy != 0 && sy == sy0) ? (double)sy : 0.5 * (vb + vt0);
          const bool wall = mr_wall(r, I.ny, I.bcy);
          if (v > 0.0 && !wall) { J += I.dx * (sb - st0); len += I.dx; }
          if (-v > 0.0 && !wall) { J0 += I.dx * (st0 - sb); len0 += I.dx; }
          /* the row below is complete */
          const int rf = r - 1;
          if (rf >= tl.y0 && cx >= 1 && cx <= KX_W - 2 && x < nx + I.fhalo) {
            const double num = fabs(J0);
            const double den = I.dx * I.dx * len0 * nrm0;
            fl[(long long)(rf + I.fhalo) * I.fex + (x + I.fhalo)] = (unsigned char)(num > den);
            if (aleph && x >= 0 && x < nx && rf >= 0 && rf < I.ny) {
              const long long cell = (long long)rf * nx + x;
              aleph[2 * cell] = num;
              aleph[2 * cell + 1] = den;
            }
          }
        }
        J0 = J; len0 = len;
      }
      nrm0 = nrm; st0 = st; vt0 = vt; sy0 = sy; act0 = act;
#pragma unroll
      for (int m = 0; m < 4; ++m) rt0[m] = rt[m];
    }
  }
}

extern "C" hipError_t mr_launch_kxrcf2_few(hipStream_t s, int nk, int bp, mr_inst* d, const mr_tile2* t, int nt,
                                           int stage) {
  if (nt <= 0) return hipSuccess;
  const dim3 G(nt), B(KX_W);
  if (nk == 3 && bp) hipLaunchKernelGGL((k2_kxrcf_few<3, true>), G, B, 0, s, d, t, nt, stage);
  else if (nk == 3) hipLaunchKernelGGL((k2_kxrcf_few<3, false>), G, B, 0, s, d, t, nt, stage);
  else if (nk == 4 && bp) hipLaunchKernelGGL((k2_kxrcf_few<4, true>), G, B, 0, s, d, t, nt, stage);
  else if (nk == 4) hipLaunchKernelGGL((k2_kxrcf_few<4, false>), G, B, 0, s, d, t, nt, stage);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}
