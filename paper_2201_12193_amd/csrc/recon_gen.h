/* Generated by gen_recon.py -- do not edit. */
#pragma once
#ifndef MR_DEV
#define MR_DEV __host__ __device__ __attribute__((always_inline))
#endif
#define MR_NKT 110
/* constants the instructions cannot encode; MR_KT(i) reads entry i
   (the including file defines MR_KT and the table storage) */
#define MR_KT_VALUES \
  0x1.0d79435e50d79p-4, 0x1.286bca1af286cp-2, 0x1.1555555555555p+0, 0x1.5555555555555p-5, \
  0x1.1745d1745d174p-4, 0x1.b45d1745d1746p+3, 0x1.d1745d1745d17p-2, 0x1.5d1745d1745d1p+3, \
  0x1.3955555555555p+0, 0x1.caaaaaaaaaaabp-4, 0x1.28e38e38e38e4p-2, 0x1.101c71c71c71dp+4, \
  0x1.f38e38e38e38ep-1, 0x1.0da12f684bda1p+1, 0x1.2025ed097b426p+5, 0x1.d12f684bda12fp+2, \
  0x1.f1c71c71c71c7p-1, 0x1.d8e38e38e38e4p+3, 0x1.11c71c71c71c7p+2, 0x1.1555555555555p+2, \
  0x1.38e6666666666p+5, 0x1.0cccccccccccdp+2, 0x1.f889249249249p+5, 0x1.38eaf8af8af8bp+9, \
  0x1.e8ef3acb2cb2dp+13, 0x1.999999999999ap-5, 0x1.47ae147ae147bp-9, 0x1.c9f25c5bfedd9p-3, \
  0x1.6e5b7d16657e1p-7, 0x1.2515fdab8464ep-11, 0x1.199999999999ap+1, 0x1.1111111111111p-6, \
  0x1.1111111111111p-5, 0x1.5555555555555p-3, 0x1.3333333333333p-1, 0x1.999999999999ap-4, \
  0x1.b26c9b26c9b27p-6, 0x1.5555555555555p-6, 0x1.d1745d1745d17p-4, 0x1.5d1745d1745d1p+1, \
  0x1.44797dd49c341p+1, 0x1.64850fe8dbd78p-5, 0x1.718966b073b4dp-4, 0x1.205c90a1fd1b8p-2, \
  0x1.1fd1b7af01724p-2, 0x1.344dd9137644ep-3, 0x1.1d79435e50d79p-4, 0x1.4b226ec89bb22p-1, \
  0x1.50d79435e50d8p-3, 0x1.b5b1e5f75270dp+0, 0x1.16c797dd49c34p-3, 0x1.2a4e1a08ad8f3p-2, \
  0x1.e115b1e5f7527p-1, 0x1.df75270d0456cp-1, 0x1.f9435e50d7943p-1, 0x1.2666666666666p-2, \
  0x1.0ad296b4a5ad3p-1, 0x1.674c59d31674cp-9, 0x1.c057d415f5058p+0, 0x1.0d79435e50d79p-5, \
  0x1.2025ed097b426p+3, 0x1.c435e50d79436p-2, 0x1.c435e50d79436p-3, 0x1.f9435e50d7943p-2, \
  0x1.c797dd49c3411p-4, 0x1.70d0456c797ddp-6, 0x1.9c34115b1e5f7p-5, 0x1.55b1e5f75270dp-3, \
  0x1.35270d0456c79p-3, 0x1.0d79435e50d79p-6, 0x1.9435e50d79436p-3, 0x1.d49c34115b1e6p-4, \
  0x1.d49c34115b1e6p-5, 0x1.d49c34115b1e6p-6, 0x1.0456c797dd49cp-6, 0x1.0456c797dd49cp-7, \
  0x1.3333333333333p-5, 0x1.3333333333333p-4, 0x1.f1c71c71c71c7p-5, 0x1.11c71c71c71c7p-2, \
  0x1.d8e38e38e38e4p-1, 0x1.0d79435e50d79p-7, 0x1.9435e50d79436p-4, 0x1.1555555555555p+3, \
  0x1.b155555555555p+5, 0x1.2aaaaaaaaaaabp+2, 0x1.5555555555555p-1, 0x1.38e6666666666p+9, \
  0x1.2d3e93e93e93fp+6, 0x1.0cccccccccccdp+5, 0x1.71c71c71c71c7p+3, 0x1.38eaf8af8af8bp+14, \
  0x1.6666666666666p+4, 0x1.2e2d82d82d82ep+10, 0x1.5389a08208208p+16, 0x1.999999999999ap-2, \
  0x1.f889249249249p+11, 0x1.a133333333333p+8, 0x1.237c57c57c57cp+8, 0x1.e8ef3acb2cb2dp+21, \
  0x1.505b6db6db6dbp+10, 0x1.53f8df545bac2p+15, 0x1.1a869536202edp+8, 0x1.52fe9ba1ba1bap+17, \
  0x1.2222222222222p+3, 0x1.52fe2be2be2bep+11, 0x1.199999999999ap+3, 0x1.999999999999ap-3, \
  0x1.c9f25c5bfedd9p-2, 0x1.0a3d70a3d70a4p-1, \
  0.0
MR_KT_DECLARE

/* modified first moment: 5/76 (u_+ - u_-) + (-11/38) (v_- + v_+) */
MR_DEV inline double mr_modified_moment(double um, double up, double vm, double vp) {
  return MR_KT(0) * (up - um) + -MR_KT(1) * (vm + vp);
}
/* ---- 1D: q_2 (3 coefs), q_3 (4), q_4 (6) of eq. (q) ---- */
MR_DEV inline void mr1_maps(double um, double u0, double up, double vm, double v0, double vp,
                            double q2[3], double q3[4], double q4[6]) {
  const double su = um + up, du = up - um, sv = vm + vp, dv = vp - vm;
  q2[0] = MR_KT(2) * u0 - MR_KT(3) * su;
  q2[1] = 0x1.0000000000000p-1 * du;
  q2[2] = -u0 + 0x1.0000000000000p-1 * su;
  q3[0] = MR_KT(2) * u0 - MR_KT(3) * su;
  q3[1] = -MR_KT(4) * du + MR_KT(5) * v0;
  q3[2] = -u0 + 0x1.0000000000000p-1 * su;
  q3[3] = MR_KT(6) * du - MR_KT(7) * v0;
  q4[0] = MR_KT(8) * u0 - MR_KT(9) * su + 0x1.b000000000000p-2 * dv;
  q4[1] = -MR_KT(10) * du + MR_KT(11) * v0 + MR_KT(12) * sv;
  q4[2] = -0x1.7000000000000p+1 * u0 + 0x1.7000000000000p+0 * su - 0x1.6800000000000p+2 * dv;
  q4[3] = MR_KT(13) * du - MR_KT(14) * v0 - MR_KT(15) * sv;
  q4[4] = 0x1.4000000000000p+0 * u0 - 0x1.4000000000000p-1 * su + 0x1.e000000000000p+1 * dv;
  q4[5] = -MR_KT(16) * du + MR_KT(17) * v0 + MR_KT(18) * sv;
}
MR_DEV inline double mr1_beta_k2(const double c[3]) {
  double b;
  { const double t = c[1];
    b = t * c[1]; }
  { const double t = MR_KT(19) * c[2];
    b = fma(t, c[2], b); }
  return b;
}
MR_DEV inline double mr1_beta_k3(const double c[4]) {
  double b;
  { const double t = c[1] + 0x1.0000000000000p-1 * c[3];
    b = t * c[1]; }
  { const double t = MR_KT(19) * c[2];
    b = fma(t, c[2], b); }
  { const double t = MR_KT(20) * c[3];
    b = fma(t, c[3], b); }
  return b;
}
MR_DEV inline double mr1_beta_k5(const double c[6]) {
  double b;
  { const double t = c[1] + 0x1.0000000000000p-1 * c[3] + 0x1.0000000000000p-3 * c[5];
    b = t * c[1]; }
  { const double t = MR_KT(19) * c[2] + MR_KT(21) * c[4];
    b = fma(t, c[2], b); }
  { const double t = MR_KT(20) * c[3] + MR_KT(22) * c[5];
    b = fma(t, c[3], b); }
  { const double t = MR_KT(23) * c[4];
    b = fma(t, c[4], b); }
  { const double t = MR_KT(24) * c[5];
    b = fma(t, c[5], b); }
  return b;
}
/* values at xi = -1/2, -sqrt(5)/10, sqrt(5)/10, 1/2 of a quintic */
MR_DEV inline void mr1_eval(const double c[6], double out[4]) {
  const double ea = c[0] + 0x1.0000000000000p-2 * c[2] + 0x1.0000000000000p-4 * c[4];
  const double oa = 0x1.0000000000000p-1 * c[1] + 0x1.0000000000000p-3 * c[3] + 0x1.0000000000000p-5 * c[5];
  const double eb = c[0] + MR_KT(25) * c[2] + MR_KT(26) * c[4];
  const double ob = MR_KT(27) * c[1] + MR_KT(28) * c[3] + MR_KT(29) * c[5];
  out[0] = ea - oa; out[1] = eb - ob; out[2] = eb + ob; out[3] = ea + oa;
}
/* ---- 2D: q_2 (6 coefs), q_3 (10), q_4 (21) of eqs. (2D-q2)-(2D-q4),
   centre average exact, other conditions in the least-squares sense.
   Monomial order: degree by degree, xi power descending:
   x^0y^0, x^1y^0, x^0y^1, x^2y^0, x^1y^1, x^0y^2, x^3y^0, x^2y^1, x^1y^2, x^0y^3, x^4y^0, x^3y^1, x^2y^2, x^1y^3, x^0y^4, x^5y^0, x^4y^1, x^3y^2, x^2y^3, x^1y^4, x^0y^5.
   With c the monomial coefficients, entry (a, b) holds 2^(1-a-b) c_ab (the
   coefficients in X = 2 xi, Y = 2 eta, twice over, so that the outer nodes are
   +-1); entries 3 and 5 hold the sum and 2/5 of the difference of the x^2 and
   y^2 coefficients, entries 10 and 14 the sum and 12/25 of the difference of
   the x^4 and y^4 ones (the exchange x <-> y decouples them) */
MR_DEV inline void mr2_maps(const double u[9], const double v[9], const double w[9],
                            double q2[6], double q3[10], double q4[21]) {
  const double ueb = u[0] + u[2];
  const double uob = u[2] - u[0];
  const double uem = u[3] + u[5];
  const double uom = u[5] - u[3];
  const double uet = u[6] + u[8];
  const double uot = u[8] - u[6];
  const double usm = u[1] + u[7];
  const double vsb = v[2] + v[0];
  const double vdb = v[2] - v[0];
  const double vsm = v[5] + v[3];
  const double vdm = v[5] - v[3];
  const double vst = v[8] + v[6];
  const double vdt = v[8] - v[6];
  const double wsl = w[6] + w[0];
  const double wdl = w[6] - w[0];
  const double wsm = w[7] + w[1];
  const double wdm = w[7] - w[1];
  const double wsr = w[8] + w[2];
  const double wdr = w[8] - w[2];
  const double vds = vdb + vdt;
  const double wds = wdl + wdr;
  const double a00 = u[4];
  const double a01 = usm + uem;
  const double a02 = usm - uem;
  const double a03 = ueb + uet;
  const double a10 = uom;
  const double a11 = uob + uot;
  const double a20 = u[7] - u[1];
  const double a21 = uet - ueb;
  const double a30 = uot - uob;
  const double b10 = vsm;
  const double b11 = vsb + vst;
  const double b12 = v[4];
  const double b20 = vdt - vdb;
  const double b30 = vst - vsb;
  const double c20 = wsm;
  const double c21 = wsl + wsr;
  const double c22 = w[4];
  const double c10 = wdr - wdl;
  const double c30 = wsr - wsl;
  const double b00 = vdm + wdm;
  const double b01 = vds + wds;
  const double c00 = vdm - wdm;
  const double c01 = vds - wds;
  q2[0] = MR_KT(30) * a00 - MR_KT(31) * a01 - MR_KT(32) * a03;
  q2[1] = MR_KT(33) * a10 + MR_KT(33) * a11;
  q2[2] = MR_KT(33) * a20 + MR_KT(33) * a21;
  q2[3] = -MR_KT(34) * a00 + MR_KT(25) * a01 + MR_KT(35) * a03;
  q2[4] = 0x1.0000000000000p-3 * a30;
  q2[5] = -MR_KT(35) * a02;
  q3[0] = MR_KT(30) * a00 - MR_KT(31) * a01 - MR_KT(32) * a03;
  q3[1] = -MR_KT(36) * a10 - MR_KT(37) * a11 + MR_KT(5) * b12;
  q3[2] = -MR_KT(36) * a20 - MR_KT(37) * a21 + MR_KT(5) * c22;
  q3[3] = -MR_KT(34) * a00 + MR_KT(25) * a01 + MR_KT(35) * a03;
  q3[4] = 0x1.0000000000000p-3 * a30;
  q3[5] = -MR_KT(35) * a02;
  q3[6] = MR_KT(38) * a10 - MR_KT(39) * b12;
  q3[7] = -0x1.0000000000000p-3 * a20 + 0x1.0000000000000p-4 * a21;
  q3[8] = -0x1.0000000000000p-3 * a10 + 0x1.0000000000000p-4 * a11;
  q3[9] = MR_KT(38) * a20 - MR_KT(39) * c22;
  q4[0] = MR_KT(40) * a00 - MR_KT(41) * a01 - MR_KT(42) * a03 + MR_KT(43) * b00 + MR_KT(44) * b01;
  q4[1] = -MR_KT(45) * a10 - MR_KT(46) * a11 + MR_KT(47) * b10 + MR_KT(48) * b11 + MR_KT(11) * b12 + 0x1.b000000000000p-3 * c10;
  q4[2] = -MR_KT(45) * a20 - MR_KT(46) * a21 + 0x1.b000000000000p-3 * b20 + MR_KT(47) * c20 + MR_KT(48) * c21 + MR_KT(11) * c22;
  q4[3] = -MR_KT(49) * a00 + MR_KT(50) * a01 + MR_KT(51) * a03 - MR_KT(52) * b00 - MR_KT(53) * b01;
  q4[4] = MR_KT(1) * a30 - MR_KT(54) * b30 - MR_KT(54) * c30;
  q4[5] = -MR_KT(55) * a02 - 0x1.8000000000000p-2 * c00 - 0x1.8000000000000p-2 * c01;
  q4[6] = MR_KT(56) * a10 + MR_KT(57) * a11 - MR_KT(58) * b10 - MR_KT(59) * b11 - MR_KT(60) * b12;
  q4[7] = -MR_KT(61) * a20 + MR_KT(62) * a21 - 0x1.6800000000000p-1 * b20 + MR_KT(54) * c20 - MR_KT(63) * c21;
  q4[8] = -MR_KT(61) * a10 + MR_KT(62) * a11 + MR_KT(54) * b10 - MR_KT(63) * b11 - 0x1.6800000000000p-1 * c10;
  q4[9] = MR_KT(56) * a20 + MR_KT(57) * a21 - MR_KT(58) * c20 - MR_KT(59) * c21 - MR_KT(60) * c22;
  q4[10] = MR_KT(64) * a00 + MR_KT(65) * a01 - MR_KT(66) * a03 + MR_KT(67) * b00 + MR_KT(68) * b01;
  q4[11] = -MR_KT(69) * a30 + MR_KT(70) * b30;
  q4[12] = MR_KT(71) * a00 - MR_KT(72) * a01 + MR_KT(73) * a03 - MR_KT(74) * b00 + MR_KT(75) * b01;
  q4[13] = -MR_KT(69) * a30 + MR_KT(70) * c30;
  q4[14] = MR_KT(76) * a02 + MR_KT(77) * c00 + MR_KT(77) * c01;
  q4[15] = -MR_KT(78) * a10 + MR_KT(79) * b10 + MR_KT(80) * b12;
  q4[16] = 0x1.4000000000000p-5 * a20 - 0x1.4000000000000p-6 * a21 + 0x1.e000000000000p-4 * b20;
  q4[17] = MR_KT(69) * a10 - MR_KT(81) * a11 - MR_KT(70) * b10 + MR_KT(82) * b11;
  q4[18] = MR_KT(69) * a20 - MR_KT(81) * a21 - MR_KT(70) * c20 + MR_KT(82) * c21;
  q4[19] = 0x1.4000000000000p-5 * a10 - 0x1.4000000000000p-6 * a11 + 0x1.e000000000000p-4 * c10;
  q4[20] = -MR_KT(78) * a20 + MR_KT(79) * c20 + MR_KT(80) * c22;
  /* 119 non-zero map entries after the parity split */
}
/* largest |coefficient| of a datum in q_l - u_5 at the face points (rounded up):
   UE, UC: averages of the edge and corner neighbours minus u_5; M0, ME, MC:
   first moments of the cell, its edge and its corner neighbours */
#define MR_BND_Q2_UE 0.14001
#define MR_BND_Q2_UC 0.26253
#define MR_BND_Q2_M0 0.00000
#define MR_BND_Q2_ME 0.00000
#define MR_BND_Q2_MC 0.00000
#define MR_BND_Q3_UE 0.08774
#define MR_BND_Q3_UC 0.13751
#define MR_BND_Q3_M0 5.45509
#define MR_BND_Q3_ME 0.00000
#define MR_BND_Q3_MC 0.00000
#define MR_BND_Q4_UE 0.25742
#define MR_BND_Q4_UC 0.34411
#define MR_BND_Q4_M0 4.46341
#define MR_BND_Q4_ME 0.58902
#define MR_BND_Q4_MC 0.96215
MR_DEV inline double mr2_beta_k2(const double c[6]) {
  double b = 0.0, part;
  { const double t = MR_KT(83) * c[3];
    part = t * c[3]; }
  b += part;
  { const double t = MR_KT(84) * c[5];
    part = t * c[5]; }
  b += part;
  { const double t = c[1];
    part = t * c[1]; }
  b += part;
  { const double t = c[2];
    part = t * c[2]; }
  b += part;
  { const double t = MR_KT(85) * c[4];
    part = t * c[4]; }
  b += part;
  return b;
}
MR_DEV inline double mr2_beta_k3(const double c[10]) {
  double b = 0.0, part;
  { const double t = MR_KT(83) * c[3];
    part = t * c[3]; }
  b += part;
  { const double t = MR_KT(84) * c[5];
    part = t * c[5]; }
  b += part;
  { const double t = c[1] + 0x1.0000000000000p+1 * c[6] + MR_KT(86) * c[8];
    part = t * c[1]; }
  { const double t = MR_KT(87) * c[6] + MR_KT(86) * c[8];
    part = fma(t, c[6], part); }
  { const double t = MR_KT(88) * c[8];
    part = fma(t, c[8], part); }
  b += part;
  { const double t = c[2] + MR_KT(86) * c[7] + 0x1.0000000000000p+1 * c[9];
    part = t * c[2]; }
  { const double t = MR_KT(88) * c[7] + MR_KT(86) * c[9];
    part = fma(t, c[7], part); }
  { const double t = MR_KT(87) * c[9];
    part = fma(t, c[9], part); }
  b += part;
  { const double t = MR_KT(85) * c[4];
    part = t * c[4]; }
  b += part;
  return b;
}
MR_DEV inline double mr2_beta_k5(const double c[21]) {
  double b = 0.0, part;
  { const double t = MR_KT(83) * c[3] + MR_KT(89) * c[10] + MR_KT(90) * c[12];
    part = t * c[3]; }
  { const double t = MR_KT(91) * c[10] + MR_KT(92) * c[12];
    part = fma(t, c[10], part); }
  { const double t = MR_KT(93) * c[12];
    part = fma(t, c[12], part); }
  b += part;
  { const double t = MR_KT(84) * c[5] + 0x1.5e00000000000p+7 * c[14];
    part = t * c[5]; }
  { const double t = MR_KT(94) * c[14];
    part = fma(t, c[14], part); }
  b += part;
  { const double t = c[1] + 0x1.0000000000000p+1 * c[6] + MR_KT(86) * c[8] + 0x1.0000000000000p+1 * c[15] + MR_KT(86) * c[17] + MR_KT(95) * c[19];
    part = t * c[1]; }
  { const double t = MR_KT(87) * c[6] + MR_KT(86) * c[8] + MR_KT(96) * c[15] + MR_KT(97) * c[17] + MR_KT(95) * c[19];
    part = fma(t, c[6], part); }
  { const double t = MR_KT(88) * c[8] + MR_KT(86) * c[15] + 0x1.2400000000000p+7 * c[17] + MR_KT(98) * c[19];
    part = fma(t, c[8], part); }
  { const double t = MR_KT(99) * c[15] + MR_KT(100) * c[17] + MR_KT(95) * c[19];
    part = fma(t, c[15], part); }
  { const double t = MR_KT(101) * c[17] + MR_KT(102) * c[19];
    part = fma(t, c[17], part); }
  { const double t = MR_KT(103) * c[19];
    part = fma(t, c[19], part); }
  b += part;
  { const double t = c[2] + MR_KT(86) * c[7] + 0x1.0000000000000p+1 * c[9] + MR_KT(95) * c[16] + MR_KT(86) * c[18] + 0x1.0000000000000p+1 * c[20];
    part = t * c[2]; }
  { const double t = MR_KT(88) * c[7] + MR_KT(86) * c[9] + MR_KT(98) * c[16] + 0x1.2400000000000p+7 * c[18] + MR_KT(86) * c[20];
    part = fma(t, c[7], part); }
  { const double t = MR_KT(87) * c[9] + MR_KT(95) * c[16] + MR_KT(97) * c[18] + MR_KT(96) * c[20];
    part = fma(t, c[9], part); }
  { const double t = MR_KT(103) * c[16] + MR_KT(102) * c[18] + MR_KT(95) * c[20];
    part = fma(t, c[16], part); }
  { const double t = MR_KT(101) * c[18] + MR_KT(100) * c[20];
    part = fma(t, c[18], part); }
  { const double t = MR_KT(99) * c[20];
    part = fma(t, c[20], part); }
  b += part;
  { const double t = MR_KT(85) * c[4] + MR_KT(104) * c[11] + MR_KT(104) * c[13];
    part = t * c[4]; }
  { const double t = MR_KT(105) * c[11] + MR_KT(106) * c[13];
    part = fma(t, c[11], part); }
  { const double t = MR_KT(105) * c[13];
    part = fma(t, c[13], part); }
  b += part;
  return b;
}
/* values of the polynomial (2D basis above; half the sum of the entries times
   the monomials in X, Y: the factor 1/2 belongs to the caller's weights) at
   (xi_k, eta_l), out[k + 4 l], xi, eta in {-1/2, -sqrt(5)/10, sqrt(5)/10, 1/2} */
MR_DEV inline void mr2_eval(const double c[21], double out[16]) {
  const double h = c[10] + c[12];
  const double e00 = c[0] + (c[3] + h);
  const double e11 = c[0] + MR_KT(107) * (c[3] + MR_KT(107) * h);
  const double em = c[0] + MR_KT(34) * c[3] + MR_KT(109) * c[10] + MR_KT(107) * c[12];
  const double ed = c[5] + c[14];
  const double e01 = em + ed;
  const double e10 = em - ed;
  const double xa = c[1] + c[6] + c[15];
  const double xb = c[1] + MR_KT(107) * (c[6] + MR_KT(107) * c[15]);
  const double xc = c[8] + c[17];
  const double xd = c[8] + MR_KT(107) * c[17];
  const double x00 = xa + (xc + c[19]);
  const double x01 = xa + MR_KT(107) * (xc + MR_KT(107) * c[19]);
  const double x10 = xb + (xd + c[19]);
  const double x11 = xb + MR_KT(107) * (xd + MR_KT(107) * c[19]);
  const double ya = c[2] + c[9] + c[20];
  const double yb = c[2] + MR_KT(107) * (c[9] + MR_KT(107) * c[20]);
  const double yc = c[7] + c[18];
  const double yd = c[7] + MR_KT(107) * c[18];
  const double y00 = ya + (yc + c[16]);
  const double y01 = ya + MR_KT(107) * (yc + MR_KT(107) * c[16]);
  const double y10 = yb + (yd + c[16]);
  const double y11 = yb + MR_KT(107) * (yd + MR_KT(107) * c[16]);
  const double g = c[11] + c[13];
  const double r00 = c[4] + g;
  const double r11 = c[4] + MR_KT(107) * g;
  const double r01 = c[4] + c[11] + MR_KT(107) * c[13];
  const double r10 = c[4] + c[13] + MR_KT(107) * c[11];
  const double s1_00 = e00 + r00;
  const double d1_00 = e00 - r00;
  const double s2_00 = x00 + y00;
  const double d2_00 = x00 - y00;
  out[0] = s1_00 - s2_00;
  out[3] = d1_00 + d2_00;
  out[12] = d1_00 - d2_00;
  out[15] = s1_00 + s2_00;
  const double s1_01 = fma(MR_KT(108), r01, e01);
  const double d1_01 = fma(-MR_KT(108), r01, e01);
  const double s2_01 = fma(MR_KT(108), y10, x01);
  const double d2_01 = fma(-MR_KT(108), y10, x01);
  out[4] = s1_01 - s2_01;
  out[7] = d1_01 + d2_01;
  out[8] = d1_01 - d2_01;
  out[11] = s1_01 + s2_01;
  const double s1_10 = fma(MR_KT(108), r10, e10);
  const double d1_10 = fma(-MR_KT(108), r10, e10);
  const double s2_10 = fma(MR_KT(108), x10, y01);
  const double d2_10 = fma(MR_KT(108), x10, -y01);
  out[1] = s1_10 - s2_10;
  out[2] = d1_10 + d2_10;
  out[13] = d1_10 - d2_10;
  out[14] = s1_10 + s2_10;
  const double s1_11 = fma(MR_KT(107), r11, e11);
  const double d1_11 = fma(-MR_KT(107), r11, e11);
  const double s2_11 = x11 + y11;
  const double d2_11 = x11 - y11;
  out[5] = fma(-MR_KT(108), s2_11, s1_11);
  out[6] = fma(MR_KT(108), d2_11, d1_11);
  out[9] = fma(-MR_KT(108), d2_11, d1_11);
  out[10] = fma(MR_KT(108), s2_11, s1_11);
}
