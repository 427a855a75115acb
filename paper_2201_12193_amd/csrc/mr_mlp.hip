/* Learned troubled-cell indicator for 2D Euler: feature extraction, the
 * fused BF16-MFMA inference kernel with its KXRCF fallback, and the kernels
 * that train the network (forward, backward, Adam).
 *
 * The indicator is not part of the paper's method: it is a small network
 * trained on the KXRCF flags (eq. (KXRCF_)) of the method's own runs, used
 * in place of Step 2.1 where it is confident.  Cells whose score falls in
 * the band [band_lo, band_hi] get the KXRCF decision.
 *
 * Features of cell (x, y): moment m in {0, 1, 2} (cell average, x and y
 * first moments) of component c in {rho, rho u, rho v, E} at cell
 * (x + wx, y + wy), |wx|, |wy| <= 2, normalised by the cell's own averages:
 *   (raw - [m == 0] centre_c) * scale_c  (evaluated as one fma with the
 *   scaled centre),
 *   scale_rho = 1/rho, scale_(rho u) = scale_(rho v) = 1/(rho c), scale_E = 1/E,
 * with c the sound speed of the cell average, plus log2(h)/16.  The values
 * are computed in FP32 and rounded to BF16.  Index of a feature: f =
 * 32 kb + 8 g + j (kb < 10, g < 4, j < 8) with slot s = 8 kb + j:
 *   s < 60:        c = s / 15, m = (s / 5) % 3, wx = s % 5 - 2, wy = g - 2;
 *   60 <= s < 75:  c = g, m = (s - 60) / 5, wx = (s - 60) % 5 - 2, wy = 2;
 *   s = 75, g = 0: log2(h)/16;   every other index is 0.
 * This order lets lane group g of the MFMA operand read window row g - 2 at
 * offsets fixed at compile time. */
#define MR_KT_IN_LDS 1
#include <algorithm>

#include "mr_common.h"
#include "mr_mlp.h"

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef short i16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

MR_INL f32x4 mr_mfma(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

/* ------------------------------------------------------------ features */
/* normalisation of a cell from its FP32 averages: scale sc[4] and the
 * scaled centre cs[c] = centre_c * sc[c] (a feature is one fma) */
MR_INL void mr_feat_norm(float rho, float mx, float my, float E, float gam, float* sc, float* cs) {
  /* hardware reciprocal and square root (1 ulp): the features are rounded
     to BF16 afterwards */
  const float r = rho > 1e-30f ? rho : 1e-30f;
  const float ir = __builtin_amdgcn_rcpf(r);
  const float p = (gam - 1.0f) * (E - 0.5f * (mx * mx + my * my) * ir);
  float c2 = gam * p * ir;
  c2 = c2 > 1e-30f ? c2 : 1e-30f;
  const float rc = __builtin_amdgcn_rcpf(r * __builtin_amdgcn_sqrtf(c2));
  sc[0] = ir;
  sc[1] = rc;
  sc[2] = rc;
  sc[3] = __builtin_amdgcn_rcpf(E > 1e-30f ? E : 1e-30f);
  cs[0] = rho * sc[0];
  cs[1] = mx * sc[1];
  cs[2] = my * sc[2];
  cs[3] = E * sc[3];
}

MR_INL float mr_feat_val(float raw, int m, float scentre, float scale) {
  return m == 0 ? fmaf(raw, scale, -scentre) : raw * scale;
}

/* slot s of lane group g -> (component, moment, wx, wy); kind 0 moment,
 * 1 log h, 2 zero */
struct mr_fslot {
  int c, m, wx, wy, kind;
};
MR_HD mr_fslot mr_feature_slot(int s, int g) {
  if (s < 60) return mr_fslot{s / 15, (s / 5) % 3, s % 5 - 2, g - 2, 0};
  if (s < 75) return mr_fslot{g, (s - 60) / 5, (s - 60) % 5 - 2, 2, 0};
  if (s == 75 && g == 0) return mr_fslot{0, 0, 0, 0, 1};
  return mr_fslot{0, 0, 0, 0, 2};
}

/* features of n interior cells (indices j*nx + i) of one instance, one
 * thread per feature; out [n][MR_KP]; an index outside the grid gives a
 * zero row */
__global__ __launch_bounds__(MR_BLOCK) void k_features(const mr_inst* insts, int inst, const int* cells, int n,
                                                      __bf16* out) {
  const long long e = (long long)blockIdx.x * MR_BLOCK + threadIdx.x;
  if (e >= (long long)n * MR_KP) return;
  const int smp = (int)(e / MR_KP), f = (int)(e % MR_KP);
  const mr_inst& I = insts[inst];
  const mr_grid g{mr_gp(I.p_in[0]), I.plane, I.nx, I.ny, I.bcx, I.bcy, 3, nullptr, 0.0};
  const int cell = cells[smp];
  if (cell < 0 || (long long)cell >= I.plane) {   /* not an interior cell */
    out[e] = (__bf16)0.0f;
    return;
  }
  const int x = cell % I.nx, y = cell / I.nx;
  const mr_fslot sl = mr_feature_slot(8 * (f / 32) + f % 8, (f / 8) % 4);
  float v = 0.0f;
  if (sl.kind == 1) {
    v = (float)(log2(I.dx) * (1.0 / 16.0));
  } else if (sl.kind == 0) {
    float sc[4], cs[4];
    mr_feat_norm((float)mr_ld(g, 0, 0, x, y), (float)mr_ld(g, 1, 0, x, y), (float)mr_ld(g, 2, 0, x, y),
                 (float)mr_ld(g, 3, 0, x, y), (float)I.gam, sc, cs);
    v = mr_feat_val((float)mr_ld(g, sl.c, sl.m, x + sl.wx, y + sl.wy), sl.m, cs[sl.c], sc[sl.c]);
  }
  out[e] = (__bf16)v;
}

/* ------------------------------------------------------------ fused inference */
/* Work item: a strip of 64 columns x `rows` rows of the extended flag range
 * [-2, n+2)^2.  The four waves of a work group take four consecutive rows
 * per sweep step; the moments of rows y-2 .. y+5 sit in an LDS ring of
 * eight FP32 rows, the next four rows' loads in flight while a step
 * computes.  Per wave and step, 64 cells in four groups of 16 (group gi:
 * cells 4 r + gi, r < 16, so that the 5-column windows of a lane's four cells
 * are eight consecutive staged columns, two 16-byte LDS reads per plane and
 * row):
 *   layer 1: h1 (64 x 16) = W1 (64 x 320) X (320 x 16), 40 MFMAs;
 *   layer 2: h2 = W2 relu(h1 + b1), 8 MFMAs, with the contraction order
 *            permuted alike on both operands so that the layer-1
 *            accumulators serve as the B operand without a transpose;
 *   layer 3: a dot product reduced across the four lane groups.
 * What bounds it: instruction issue.  Of the time at 2048 x 2048 the 304
 * multiplications that scale a wave's features and their 152 conversions
 * take 20 %, the matrix instructions of layer 1 18 %, staging 12 %, those of
 * layer 2 4 %, the norms 3 %; HBM would allow 100 us.  Deeper rings with one
 * barrier a step or none, eight-wave groups and raised wave priorities
 * measured the same or slower.  118 -> 77 us at 1024 x 1024; 333 -> 295
 * us at 2048 x 2048 with the fallback below (windows read 16 bytes at a
 * time, loads a step ahead, vector work behind each matrix instruction, the
 * undecided cells gathered in LDS, the strips' height).
 * Lane i of the MFMA holds A[i%16][8(i/16)+j], B[8(i/16)+j][i%16] (j < 8)
 * and receives D[4(i/16)+j][i%16] (j < 4). */
#define MR_LW 64                       /* cells per strip row              */
#define MR_LCOLS (MR_LW + 4)           /* staged columns                   */
#define MR_LRS MR_LCOLS                /* LDS row stride (floats)          */
#define MR_LPL (8 * MR_LRS + 16)       /* LDS plane stride (floats)        */
#define MR_LBAND 1408                  /* undecided cells held in LDS      */
struct __attribute__((aligned(16))) mr_learn_lds {
  mr_learn_w w;
  float mom[12 * MR_LPL];
  int nband, base;                     /* cells in the list; its place in the band */
  unsigned short band[MR_LBAND];       /* 64 (row in the strip) + column    */
};

/* eight consecutive floats of LDS, 16-byte aligned */
MR_INL void mr_ld8f(const float* p, float v[8]) {
  const float4 a = reinterpret_cast<const float4*>(p)[0], b = reinterpret_cast<const float4*>(p)[1];
  v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
  v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}

__global__ __launch_bounds__(MR_BLOCK, 2) void k2_learned(const mr_inst* __restrict__ insts, const mr_tile2* __restrict__ tiles, int ntiles,
                                                         int stage, const mr_learn_w* wg, mr_band* band, int* cnt) {
  __shared__ mr_learn_lds sh;
  const int tid = threadIdx.x, lane = tid % 64, wv = tid / 64, r = lane % 16, g = lane / 16;
  {
    const uint4* src = reinterpret_cast<const uint4*>(wg);
    uint4* dst = reinterpret_cast<uint4*>(&sh.w);
    for (int e = tid; e < (int)(sizeof(mr_learn_w) / 16); e += MR_BLOCK) dst[e] = src[e];
  }
  const bf16x8* W1 = reinterpret_cast<const bf16x8*>(sh.w.w1);
  const bf16x8* W2 = reinterpret_cast<const bf16x8*>(sh.w.w2);
  /* staging: thread (column scol, moment sm) of the first 3 x 68 threads
     loads that column and moment of every component and row */
  const int scol = tid % MR_LCOLS, sm = tid / MR_LCOLS;
  const bool stager = tid < 3 * MR_LCOLS;
  for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
    const mr_tile2 tl = tiles[t];
    const mr_inst& I = insts[tl.inst];
    if (stage < 3 && !I.active) continue;
    if (I.tc != 3) continue;
    const mr_grid gr{mr_gp(stage < 3 ? I.p_in[stage] : I.buf[0]), I.plane, I.nx, I.ny, I.bcx, I.bcy, 3, nullptr, 0.0};
    MR_GLB unsigned char* fl = mr_gp(I.flags[(stage == 0 || stage == 3) ? 0 : 1]);
    const int fh = I.fhalo, fex = I.fex;
    const int xs = tl.x0 - 2, ylo = tl.y0, yhi = tl.y0 + tl.rows;
    const int xend = I.nx + fh;
    const float gam = (float)I.gam, lh = (float)(log2(I.dx) * (1.0 / 16.0));
    const float blo = (float)I.band_lo, bhi = (float)I.band_hi;
    /* staging of four rows: every thread issues its loads together, into
       registers; they are converted and stored later.  First moments of
       transmissive ghosts read as zero, reflective ghosts flip the moments
       mr_refl_flip names; strips and rows without ghosts skip those rules */
    int kx = 0;
    const int ii = mr_fold(xs + scol, I.nx, I.bcx, &kx);
    const bool xplain = (xs >= 0 || (I.bcx & 3) == 0) && (xs + MR_LCOLS <= I.nx || ((I.bcx >> 2) & 3) == 0);
    const long long P = I.plane;
    const MR_GLB double* ub = gr.U + (long long)sm * P + ii;
    double pf[16];
    int kys = 0;   /* y ghost kind of row rr in bits 2 rr, 2 rr + 1 (uniform) */
    auto fetch = [&](int row0) {
      kys = 0;
#pragma unroll
      for (int rr = 0; rr < 4; ++rr) {
        int ky = 0;
        const long long jj = (long long)mr_fold(row0 + rr, I.ny, I.bcy, &ky) * I.nx;
        kys |= ky << (2 * rr);
        if (stager) {
#pragma unroll
          for (int c = 0; c < 4; ++c) pf[4 * rr + c] = (ub + (3 * c) * P)[jj];
        }
      }
    };
    auto store = [&](int row0) {
      if (!stager) return;
#pragma unroll
      for (int rr = 0; rr < 4; ++rr) {
        const int slot = (row0 + rr - ylo + 2) & 7;
        float* d = sh.mom + sm * MR_LPL + slot * MR_LRS + scol;
        if (xplain && kys == 0) {
#pragma unroll
          for (int c = 0; c < 4; ++c) d[3 * c * MR_LPL] = (float)pf[4 * rr + c];
        } else {
          const int ky = (kys >> (2 * rr)) & 3;
          const bool zero = sm != 0 && (kx == 1 || ky == 1);
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            const bool neg = (kx == 2 && mr_refl_flip(c, sm, 0)) != (ky == 2 && mr_refl_flip(c, sm, 1));
            const double v = pf[4 * rr + c];
            d[3 * c * MR_LPL] = (float)(zero ? 0.0 : (neg ? -v : v));
          }
        }
      }
    };
    __syncthreads();
    if (tid == 0) sh.nband = 0;
    fetch(ylo - 2);
    store(ylo - 2);   /* rows ylo-2 .. ylo+1 */
    fetch(ylo + 2);
    store(ylo + 2);   /* rows ylo+2 .. ylo+5 */
    __syncthreads();
    for (int y = ylo; y < yhi; y += 4) {
      const bool more = y + 4 < yhi;
      if (more) fetch(y + 6);   /* the rows that replace y-2 .. y+1 */
      const int Y = y + wv;
      /* LDS bases (16-byte aligned): centre row, the lane group's window row
         (wy = g - 2), and window row wy = 2 of component g */
      const int bc = ((Y - ylo + 2) & 7) * MR_LRS + 4 * r;
      const int bo = ((Y - ylo + g) & 7) * MR_LRS + 4 * r;
      const int b2 = ((Y - ylo + 4) & 7) * MR_LRS + 4 * r + 3 * g * MR_LPL;
      float sc[4][4], cs[4][4], scg[4], csg[4];
      {
        float ctr[4][8];
#pragma unroll
        for (int c = 0; c < 4; ++c) mr_ld8f(&sh.mom[3 * c * MR_LPL + bc], ctr[c]);
#pragma unroll
        for (int gi = 0; gi < 4; ++gi)
          mr_feat_norm(ctr[0][gi + 2], ctr[1][gi + 2], ctr[2][gi + 2], ctr[3][gi + 2], gam, sc[gi], cs[gi]);
      }
#pragma unroll
      for (int gi = 0; gi < 4; ++gi) {
        scg[gi] = g == 0 ? sc[gi][0] : (g == 3 ? sc[gi][3] : sc[gi][1]);
        csg[gi] = g == 0 ? cs[gi][0] : (g == 1 ? cs[gi][1] : (g == 2 ? cs[gi][2] : cs[gi][3]));
      }
      /* the accumulators start from the biases: lane (r, g) accumulates
         hidden units 16m + 4g + j */
      const float4* b1v4 = reinterpret_cast<const float4*>(sh.w.b1);
      const float4* b2v4 = reinterpret_cast<const float4*>(sh.w.b2);
      const float4* w3v4 = reinterpret_cast<const float4*>(sh.w.w3);
      f32x4 h[4][4];
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const float4 bb = b1v4[4 * m + g];
#pragma unroll
        for (int gi = 0; gi < 4; ++gi) h[gi][m] = f32x4{bb.x, bb.y, bb.z, bb.w};
      }
      /* planes of the window, five slots each: plane p < 12 moment p of the
         lane's own row, p = 12 .. 14 moment p - 12 of component g in row
         wy = 2 */
      float rw[15][8];
      auto plane = [&](int p) { mr_ld8f(&sh.mom[p < 12 ? p * MR_LPL + bo : (p - 12) * MR_LPL + b2], rw[p]); };
      auto feat = [&](int s, int gi) -> float {
        if (s < 60) return mr_feat_val(rw[s / 5][s % 5 + gi], (s / 5) % 3, cs[gi][s / 15], sc[gi][s / 15]);
        if (s < 75) return mr_feat_val(rw[s / 5][s % 5 + gi], (s - 60) / 5, csg[gi], scg[gi]);
        return s == 75 && g == 0 ? lh : 0.0f;
      };
      /* layer 1, pipelined by hand: behind each matrix instruction the vector
         instructions of two features of the next operand, which run while it
         occupies the matrix core (in the compiler's order, four matrix
         instructions and then twelve vector ones, the two hardly overlap);
         weights and planes are read a contraction block ahead */
      bf16x8 a[2][4], b;
#pragma unroll
      for (int m = 0; m < 4; ++m) a[0][m] = W1[m * 64 + lane];
      plane(0);
      plane(1);
#pragma unroll
      for (int j = 0; j < 8; ++j) b[j] = (__bf16)feat(j, 0);
#pragma unroll
      for (int kb = 0; kb < MR_KP / 32; ++kb) {
        if (kb + 1 < MR_KP / 32) {
#pragma unroll
          for (int m = 0; m < 4; ++m) a[(kb + 1) & 1][m] = W1[((kb + 1) * 4 + m) * 64 + lane];
#pragma unroll
          for (int p = 2; p < 15; ++p)
            if (p > (8 * kb + 7) / 5 && p <= (8 * kb + 15) / 5) plane(p);
        }
#pragma unroll
        for (int gi = 0; gi < 4; ++gi) {
          const int nk = kb + (gi == 3), ng = (gi + 1) & 3;
          bf16x8 bn = {};
#pragma unroll
          for (int m = 0; m < 4; ++m) {
            h[gi][m] = mr_mfma(a[kb & 1][m], b, h[gi][m]);
            if (nk < MR_KP / 32) {
              const bf16x2 f2 = __builtin_convertvector(f32x2{feat(8 * nk + 2 * m, ng), feat(8 * nk + 2 * m + 1, ng)}, bf16x2);
              bn[2 * m] = f2[0];
              bn[2 * m + 1] = f2[1];
            }
            __builtin_amdgcn_sched_barrier(0);
          }
          b = bn;
        }
      }
      /* layer 2 and 3; this lane holds hidden units 16m + 4g + j */
      bf16x8 a2[2][4];
      float4 b2v[4], w3v[4];
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        a2[0][m] = W2[m * 64 + lane];
        a2[1][m] = W2[(4 + m) * 64 + lane];
        b2v[m] = b2v4[4 * m + g];
        w3v[m] = w3v4[4 * m + g];
      }
      float z[4];
#pragma unroll
      for (int gi = 0; gi < 4; ++gi) {
        f32x4 o[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) o[m] = f32x4{b2v[m].x, b2v[m].y, b2v[m].z, b2v[m].w};
#pragma unroll
        for (int kb2 = 0; kb2 < 2; ++kb2) {
          const f32x4 x = h[gi][2 * kb2], y = h[gi][2 * kb2 + 1];
          const bf16x2 p0 = __builtin_convertvector(f32x2{x[0], x[1]}, bf16x2);
          const bf16x2 p1 = __builtin_convertvector(f32x2{x[2], x[3]}, bf16x2);
          const bf16x2 p2 = __builtin_convertvector(f32x2{y[0], y[1]}, bf16x2);
          const bf16x2 p3 = __builtin_convertvector(f32x2{y[2], y[3]}, bf16x2);
          bf16x8 bb = {p0[0], p0[1], p1[0], p1[1], p2[0], p2[1], p3[0], p3[1]};
          /* ReLU after the rounding (rounding keeps the sign): a negative
             BF16 is a negative int16, so a packed integer max with 0 clears
             it, two values per instruction */
          bb = __builtin_bit_cast(bf16x8, __builtin_elementwise_max(__builtin_bit_cast(i16x8, bb), i16x8{}));
#pragma unroll
          for (int m = 0; m < 4; ++m) o[m] = mr_mfma(a2[kb2][m], bb, o[m]);
        }
        float zp = 0.f;
#pragma unroll
        for (int m = 0; m < 4; ++m) {
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const float v = o[m][j];
            /* ReLU on the bit pattern: a negative float is a negative int32 */
            zp += __builtin_bit_cast(float, max(__builtin_bit_cast(int, v), 0)) * (&w3v[m].x)[j];
          }
        }
        zp += __shfl_xor(zp, 16);
        zp += __shfl_xor(zp, 32);
        z[gi] = zp + sh.w.b3;
      }
      /* lane (r, g) decides cell x0 + 4 r + g of row Y */
      const float zz = g == 0 ? z[0] : (g == 1 ? z[1] : (g == 2 ? z[2] : z[3]));
      const float sg = __builtin_amdgcn_rcpf(1.0f + __expf(-zz));
      const int x = tl.x0 + 4 * r + g;
      const bool valid = Y < yhi && x < xend;
      const unsigned char f = sg > bhi ? 1 : (sg < blo ? 0 : 2);
      const long long e = (long long)(Y + fh) * fex + (x + fh);
      if (valid) fl[e] = f;
      const unsigned long long bm = __ballot(valid && f == 2);
      if (bm) {
        int base = 0;
        if (lane == 0) base = atomicAdd(&sh.nband, __popcll(bm));
        base = __shfl(base, 0);
        if (valid && f == 2)
          sh.band[base + __popcll(bm & ((1ull << lane) - 1ull))] = (unsigned short)(64 * (Y - ylo) + 4 * r + g);
      }
      __syncthreads();   /* rows y-2 .. y+1 are consumed, the list is whole */
      /* the list goes out when the next step may not fit, and at the end: one
         global atomic a strip, not one (and its round trip) a wave and row */
      if (!more || sh.nband > MR_LBAND - 4 * MR_LW) {
        const int n = sh.nband;
        if (tid == 0 && n > 0) sh.base = atomicAdd(&cnt[stage], n);
        __syncthreads();
        for (int k = tid; k < n; k += MR_BLOCK) {
          const int b = sh.band[k];
          band[sh.base + k] = mr_band{tl.inst, (int)((long long)(ylo + b / 64 + fh) * fex + (tl.x0 + b % 64 + fh))};
        }
        if (tid == 0) sh.nband = 0;
      }
      if (more) {
        store(y + 6);
        __syncthreads();
      }
    }
  }
}

/* KXRCF for the cells the network left undecided (band list, count
 * cnt[stage]) in one pass: fifteen threads per band cell reconstruct the
 * density and the momenta of the cell and of its four neighbours, five of
 * them form the face data (means and normal velocities on the four faces and
 * the norm, eqs. (line-integral-average_)), and the first evaluates eq.
 * (KXRCF_) on it as the fused indicator kernel does.  The list is short
 * (thousands of cells), so the launch lasts as long as one group's chain of
 * loads and Step 1: 21 -> 13 us at 1024 x 1024 with the components on three
 * threads, where one took them in turn, and the constant table in LDS.
 * (Deciding the velocities' signs from bounds first, five threads a cell,
 * makes the chain longer: 16 us.)
 * One launch per smoothness-indicator variant; each skips the other's cells.
 * The learned indicator takes no per-side boundary data (the library
 * rejects the combination), so its grids carry no instance for prescribed
 * ghosts. */
template <bool BP>
__global__ __launch_bounds__(MR_BLOCK) MR_OCC void k_fb_direct(const mr_inst* __restrict__ insts, const mr_band* band, const int* cnt,
                                                              int stage) {
  mr_kt_fill();
  constexpr int PB = MR_BLOCK / 15;   /* band cells per block pass */
  __shared__ double pr[PB][5][12];    /* density at points 0,4,8,12 | 3,7,11,15 | 1,2,13,14 */
  __shared__ double pm[PB][5][2][8];  /* x momentum left | right, y momentum bottom | top   */
  __shared__ double fs[PB][5][9];     /* face averages, velocities, norm                     */
  const int n = cnt[stage];
  const int tid = threadIdx.x, cb = tid / 15, d = (tid % 15) / 3, c = tid % 3;
  for (int base = blockIdx.x * PB; base < n; base += gridDim.x * PB) {
    const int k = base + cb;
    mr_band b{0, 0};
    bool mine = false;
    if (tid < 15 * PB && k < n) {
      b = band[k];
      const mr_inst& I = insts[b.inst];
      mine = (I.beta_on != 0) == BP;
      if (mine) {
        const int i = b.e % I.fex - I.fhalo, j = b.e / I.fex - I.fhalo;
        const int di = d == 1 ? -1 : (d == 2 ? 1 : 0), dj = d == 3 ? -1 : (d == 4 ? 1 : 0);
        const mr_grid g{mr_gp(stage < 3 ? I.p_in[stage] : I.buf[0]), I.plane, I.nx, I.ny, I.bcx, I.bcy, 3, nullptr, 0.0};
        double u[9], v[9], w[9], r[16];
        mr2_stencil(g, c, i + di, j + dj, u, v, w);
        mr_recon2d<BP>(u, v, w, I.W, r);
        if (c == 0) {
          double sl = 0.0, sr = 0.0, sb = 0.0, st = 0.0, nrm = 0.0;
#pragma unroll
          for (int m = 0; m < 4; ++m) {
            sl += glw(m) * r[0 + 4 * m];
            sr += glw(m) * r[3 + 4 * m];
            sb += glw(m) * r[m];
            st += glw(m) * r[12 + m];
            pr[cb][d][m] = r[4 * m];
            pr[cb][d][4 + m] = r[3 + 4 * m];
          }
          pr[cb][d][8] = r[1]; pr[cb][d][9] = r[2]; pr[cb][d][10] = r[13]; pr[cb][d][11] = r[14];
#pragma unroll
          for (int q = 0; q < 16; ++q) nrm = fmax(nrm, fabs(r[q]));
          fs[cb][d][0] = sl; fs[cb][d][1] = sr; fs[cb][d][2] = sb; fs[cb][d][3] = st; fs[cb][d][8] = nrm;
        } else {
#pragma unroll
          for (int m = 0; m < 4; ++m) {
            pm[cb][d][c - 1][m] = c == 1 ? r[4 * m] : r[m];
            pm[cb][d][c - 1][4 + m] = c == 1 ? r[3 + 4 * m] : r[12 + m];
          }
        }
      }
    }
    __syncthreads();
    if (mine && c == 0) {
      const double* q = pr[cb][d];
      const double* mx = pm[cb][d][0];
      const double* my = pm[cb][d][1];
      double irl[4], irr[4], irm[4];
      mr_recip4(q[0], q[1], q[2], q[3], irl);
      mr_recip4(q[4], q[5], q[6], q[7], irr);
      mr_recip4(q[8], q[9], q[10], q[11], irm);
      double vl = 0.0, vr = 0.0;
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        vl += glw(m) * (mx[m] * irl[m]);
        vr += glw(m) * (mx[4 + m] * irr[m]);
      }
      fs[cb][d][4] = vl;
      fs[cb][d][5] = vr;
      fs[cb][d][6] = glw(0) * (my[0] * irl[0]) + glw(1) * (my[1] * irm[0]) + glw(2) * (my[2] * irm[1]) + glw(3) * (my[3] * irr[0]);
      fs[cb][d][7] = glw(0) * (my[4] * irl[3]) + glw(1) * (my[5] * irm[2]) + glw(2) * (my[6] * irm[3]) + glw(3) * (my[7] * irr[3]);
    }
    __syncthreads();
    if (mine && c == 0 && d == 0) {
#pragma clang fp contract(off)
      const mr_inst& I = insts[b.inst];
      MR_GLB unsigned char* fl = mr_gp(I.flags[(stage == 0 || stage == 3) ? 0 : 1]);
      const int i = b.e % I.fex - I.fhalo, j = b.e / I.fex - I.fhalo;
      const double tb = mr_stage_time(I, stage);
      /* face data of a cell: 0..3 face averages (left, right, bottom, top),
         4..7 the normal velocities there, 8 the norm of its values */
      const double* o = fs[cb][0];
      const double* l = fs[cb][1];
      const double* r = fs[cb][2];
      const double* bo = fs[cb][3];
      const double* t = fs[cb][4];
      double J = 0.0, len = 0.0;
      const double vl = 0.5 * (o[4] + l[5]);
      if (vl > 0.0 && !mr_wall_x(I, i, j, tb)) { J += I.dy * (o[0] - l[1]); len += I.dy; }
      const double vr = 0.5 * (o[5] + r[4]);
      if (-vr > 0.0 && !mr_wall_x(I, i + 1, j, tb)) { J += I.dy * (o[1] - r[0]); len += I.dy; }
      const double vb = 0.5 * (o[6] + bo[7]);
      if (vb > 0.0 && !mr_wall_y(I, i, j, tb)) { J += I.dx * (o[2] - bo[3]); len += I.dx; }
      const double vt = 0.5 * (o[7] + t[6]);
      if (-vt > 0.0 && !mr_wall_y(I, i, j + 1, tb)) { J += I.dx * (o[3] - t[2]); len += I.dx; }
      fl[b.e] = (unsigned char)(fabs(J) > I.dx * I.dx * len * o[8]);
    }
    __syncthreads();
  }
}

/* before a step (stages 0..2) or a probe (stage 3): clear the band counts
 * of those stages */
__global__ void k_fb_reset(int* cnt, int probe) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  if (probe) cnt[3] = 0;
  else cnt[0] = cnt[1] = cnt[2] = 0;
}

/* BF16 parameter vector -> operand-ordered weights of the fused kernel */
__global__ void k_pack_weights(const __bf16* P, mr_learn_w* w) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e < MR_FRAG1) {
    const int lane = e % 64, m = (e / 64) % 4, kb = e / 256, r = lane % 16, g = lane / 16;
    bf16x8 v;
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = P[MR_OFF_W1 + (16 * m + r) * MR_KP + 32 * kb + 8 * g + j];
    reinterpret_cast<bf16x8*>(w->w1)[e] = v;
  } else if (e < MR_FRAG1 + MR_FRAG2) {
    const int k = e - MR_FRAG1;
    const int lane = k % 64, m = (k / 64) % 4, kb2 = k / 256, r = lane % 16, g = lane / 16;
    bf16x8 v;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      v[j] = P[MR_OFF_W2 + (16 * m + r) * MR_NH + 32 * kb2 + 4 * g + j];
      v[4 + j] = P[MR_OFF_W2 + (16 * m + r) * MR_NH + 32 * kb2 + 16 + 4 * g + j];
    }
    reinterpret_cast<bf16x8*>(w->w2)[k] = v;
  } else if (e < MR_FRAG1 + MR_FRAG2 + MR_NH) {
    const int o = e - MR_FRAG1 - MR_FRAG2;
    w->b1[o] = (float)P[MR_OFF_B1 + o];
    w->b2[o] = (float)P[MR_OFF_B2 + o];
    w->w3[o] = (float)P[MR_OFF_W3 + o];
    if (o == 0) {
      w->b3 = (float)P[MR_OFF_B3];
      w->pad[0] = w->pad[1] = w->pad[2] = 0.0f;
    }
  }
}

/* ------------------------------------------------------------ training */
/* C[m][n] = sum_k A[m][k] B[k][n] over BF16 operands with arbitrary strides,
 * FP32 accumulation; one wave per 16 x 16 tile of C. */
__global__ __launch_bounds__(MR_BLOCK) void k_gemm_bf16(int M, int N, int K, const __bf16* A, long long sAm,
                                                       long long sAk, const __bf16* B, long long sBk, long long sBn,
                                                       float* C, long long sCm, long long sCn) {
  const int tilesN = (N + 15) / 16;
  const int tile = blockIdx.x * (MR_BLOCK / 64) + threadIdx.x / 64;
  if (tile >= ((M + 15) / 16) * tilesN) return;
  const int m0 = (tile / tilesN) * 16, n0 = (tile % tilesN) * 16;
  const int lane = threadIdx.x % 64, r = lane % 16, g = lane / 16;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int k0 = 0; k0 < K; k0 += 32) {
    bf16x8 a, b;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int k = k0 + 8 * g + j;
      const bool kin = k < K;
      a[j] = (kin && m0 + r < M) ? A[(long long)(m0 + r) * sAm + (long long)k * sAk] : (__bf16)0.0f;
      b[j] = (kin && n0 + r < N) ? B[(long long)k * sBk + (long long)(n0 + r) * sBn] : (__bf16)0.0f;
    }
    acc = mr_mfma(a, b, acc);
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int m = m0 + 4 * g + j, n = n0 + r;
    if (m < M && n < N) C[(long long)m * sCm + (long long)n * sCn] = acc[j];
  }
}

/* eight consecutive BF16 values; AL: the address is 16-byte aligned */
template <bool AL>
MR_INL bf16x8 mr_ld8(const __bf16* p) {
  if (AL) return *reinterpret_cast<const bf16x8*>(p);
  bf16x8 v;
#pragma unroll
  for (int j = 0; j < 8; ++j) v[j] = p[j];
  return v;
}

/* Forward pass of 16 samples per wave (one wave per work group, so that a
 * batch of 4096 reaches every CU): h1 = relu(X W1^T + b1), h2 = relu(h1 W2^T +
 * b2), z = W3 h2 + b3, each layer handed to the next through LDS.  Operand A
 * is the samples' rows and operand B the weights' rows, both read as 16-byte
 * pieces; the contraction runs over K in order, as does the sum for z.  What
 * bounds it is the latency of one wave's chain (loads, 40 + 8 matrix
 * instructions, 64 additions): 8 us at 4096 samples, where five launches
 * with scalar operand loads took 41. */
template <bool AL>
__global__ __launch_bounds__(64) void k_mlp_fwd(int Bn, const __bf16* X, const __bf16* P, float* h1g, __bf16* h1bg,
                                                float* h2g, float* zc, float* z) {
  __shared__ __align__(16) __bf16 hb[16][MR_NH + 8];
  __shared__ float h2s[16][MR_NH + 1];
  const int lane = threadIdx.x, r = lane % 16, g = lane / 16, s0 = blockIdx.x * 16;
  const __bf16* xr = X + (long long)min(s0 + r, Bn - 1) * MR_KP + 8 * g;
  const __bf16* w1 = P + MR_OFF_W1 + r * MR_KP + 8 * g;
  f32x4 acc[4] = {};
#pragma unroll
  for (int kb = 0; kb < MR_KP / 32; ++kb) {
    const bf16x8 a = mr_ld8<AL>(xr + 32 * kb);
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) acc[nt] = mr_mfma(a, mr_ld8<AL>(w1 + 16 * nt * MR_KP + 32 * kb), acc[nt]);
  }
#pragma unroll
  for (int nt = 0; nt < 4; ++nt) {
    const int u = 16 * nt + r;
    const float b = (float)P[MR_OFF_B1 + u];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      float v = acc[nt][j] + b;
      v = v > 0.f ? v : 0.f;
      const int s = s0 + 4 * g + j;
      hb[4 * g + j][u] = (__bf16)v;
      if (s < Bn) {
        h1g[(long long)s * MR_NH + u] = v;
        h1bg[(long long)s * MR_NH + u] = (__bf16)v;
      }
    }
  }
  __syncthreads();
  const __bf16* w2 = P + MR_OFF_W2 + r * MR_NH + 8 * g;
  f32x4 ac2[4] = {};
#pragma unroll
  for (int kb = 0; kb < MR_NH / 32; ++kb) {
    const bf16x8 a = *reinterpret_cast<const bf16x8*>(&hb[r][32 * kb + 8 * g]);
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) ac2[nt] = mr_mfma(a, mr_ld8<AL>(w2 + 16 * nt * MR_NH + 32 * kb), ac2[nt]);
  }
#pragma unroll
  for (int nt = 0; nt < 4; ++nt) {
    const int u = 16 * nt + r;
    const float b = (float)P[MR_OFF_B2 + u];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      float v = ac2[nt][j] + b;
      v = v > 0.f ? v : 0.f;
      const int s = s0 + 4 * g + j;
      h2s[4 * g + j][u] = v;
      if (s < Bn) h2g[(long long)s * MR_NH + u] = v;
    }
  }
  __syncthreads();
  if (lane < 16 && s0 + lane < Bn) {
    float a = 0.0f;
    for (int o = 0; o < MR_NH; ++o) a += (float)P[MR_OFF_W3 + o] * h2s[lane][o];
    a += (float)P[MR_OFF_B3];
    zc[s0 + lane] = a;
    z[s0 + lane] = a;
  }
}

/* Backward pass of the binary cross-entropy on the logit, in chunks of
 * MR_BC samples, a work group taking chunks blockIdx.x, + gridDim.x, ..:
 *   dz = (sigmoid(z) - y) / B and the loss of each sample,
 *   d2 = dz W3 [h2 > 0] and d1 = (d2 W2) [h1 > 0], both rounded to BF16,
 *   dW2 = d2^T h1, dW1 = d1^T X, db2 = sum dz W3 [h2 > 0],
 *   dW3 = sum dz h2, db3 = sum dz, db1 = sum (d2 W2) [h1 > 0] (FP32 sums).
 * A wave forms d2 and d1 of 16 samples in registers; d2, d1, h1 and X of the
 * chunk are laid out in LDS unit by unit (samples contiguous, two per 32-bit
 * write), which makes both operands of the weight gradients 16-byte reads.
 * Wave w accumulates rows 16 w .. 16 w + 15 of dW1 and dW2 (24 tiles in
 * registers) over its group's chunks and writes them as one partial gradient
 * into part[blockIdx.x]; k_grad_sum adds the partials in order, so the
 * result does not depend on timing.  Before, the contraction over the batch
 * ran in one chain per tile with two-byte loads, and the column sums in a
 * single work group: 960 us a pass at 4096 samples, now 21 + 4. */
#define MR_BC 64                  /* samples per chunk            */
#define MR_BS (MR_BC + 8)         /* LDS row stride (samples)     */
struct mr_bwd_lds {
  __bf16 w2t[MR_NH][MR_NH + 8];   /* W2 transposed: [input unit][output unit] */
  __bf16 d2t[MR_NH][MR_BS], d1t[MR_NH][MR_BS], h1t[MR_NH][MR_BS];
  __bf16 xt[MR_KP][MR_BS];
  float dz[MR_BC];
  float red[4][4][MR_NH];
};
template <bool AL>
__global__ __launch_bounds__(256) void k_mlp_bwd(int Bn, const __bf16* X, const __bf16* P, const float* zc,
                                                 const float* y, const float* h1g, const __bf16* h1bg,
                                                 const float* h2g, float* loss, float* part) {
  __shared__ __align__(16) mr_bwd_lds sh;
  const int tid = threadIdx.x, lane = tid % 64, w = tid / 64, r = lane % 16, g = lane / 16;
  for (int e = tid; e < MR_NH * MR_NH; e += 256) sh.w2t[e % MR_NH][e / MR_NH] = P[MR_OFF_W2 + e];
  f32x4 a2[4] = {}, a1[MR_KP / 16] = {};
  float sb1[4] = {0.f, 0.f, 0.f, 0.f}, sb2 = 0.f, sw3 = 0.f, sb3 = 0.f;
  const int co = tid % MR_NH;     /* column of the FP32 sums; wave w takes its own samples */
  const float cw3 = (float)P[MR_OFF_W3 + co];
  const int nch = (Bn + MR_BC - 1) / MR_BC;
  for (int c = blockIdx.x; c < nch; c += gridDim.x) {
    const int base = c * MR_BC;
    __syncthreads();   /* the previous chunk's operands are consumed (and w2t is there) */
    /* X and h1, two samples by eight units per thread and turn */
    for (int e = tid; e < (MR_KP + MR_NH) / 8 * (MR_BC / 2); e += 256) {
      const int sp = e % (MR_BC / 2), oc = e / (MR_BC / 2), s = base + 2 * sp;
      const bool x = oc < MR_KP / 8;
      const __bf16* src = x ? X + (long long)s * MR_KP + 8 * oc : h1bg + (long long)s * MR_NH + 8 * (oc - MR_KP / 8);
      bf16x8 u = {}, v = {};
      if (s < Bn) u = mr_ld8<AL>(src);
      if (s + 1 < Bn) v = mr_ld8<AL>(src + (x ? MR_KP : MR_NH));
      __bf16* dst = x ? &sh.xt[8 * oc][2 * sp] : &sh.h1t[8 * (oc - MR_KP / 8)][2 * sp];
#pragma unroll
      for (int j = 0; j < 8; ++j) *reinterpret_cast<bf16x2*>(dst + j * MR_BS) = bf16x2{u[j], v[j]};
    }
    /* dz and d2 of sample r of the wave: operand A of d2 W2 */
    const int s = base + 16 * w + r;
    const bool in = s < Bn;
    float d = 0.f;
    if (in) {
      const float zz = zc[s], yy = y[s];
      d = (1.0f / (1.0f + expf(-zz)) - yy) / (float)Bn;
      if (g == 0) loss[s] = log1pf(expf(-fabsf(zz))) + fmaxf(zz, 0.f) - yy * zz;
    }
    if (g == 0) sh.dz[16 * w + r] = d;
    f32x4 t1[4] = {};
#pragma unroll
    for (int kb = 0; kb < MR_NH / 32; ++kb) {
      bf16x8 a = {};
      if (in) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const int o = 32 * kb + 8 * g + j;
          a[j] = (__bf16)(h2g[(long long)s * MR_NH + o] > 0.f ? d * (float)P[MR_OFF_W3 + o] : 0.f);
        }
      }
#pragma unroll
      for (int j = 0; j < 8; ++j) sh.d2t[32 * kb + 8 * g + j][16 * w + r] = a[j];
#pragma unroll
      for (int nt = 0; nt < 4; ++nt)
        t1[nt] = mr_mfma(a, *reinterpret_cast<const bf16x8*>(&sh.w2t[16 * nt + r][32 * kb + 8 * g]), t1[nt]);
    }
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
      bf16x2 lo, hi;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int sj = base + 16 * w + 4 * g + j;
        const float v = sj < Bn && h1g[(long long)sj * MR_NH + 16 * nt + r] > 0.f ? t1[nt][j] : 0.f;
        sb1[nt] += v;
        if (j < 2) lo[j] = (__bf16)v;
        else hi[j - 2] = (__bf16)v;
      }
      *reinterpret_cast<bf16x2*>(&sh.d1t[16 * nt + r][16 * w + 4 * g]) = lo;
      *reinterpret_cast<bf16x2*>(&sh.d1t[16 * nt + r][16 * w + 4 * g + 2]) = hi;
    }
    __syncthreads();
    /* FP32 column sums of column co over the wave's samples */
    for (int q = 0; q < 16; ++q) {
      const int sq = base + 16 * w + q;
      if (sq >= Bn) break;
      const float dq = sh.dz[16 * w + q], hv = h2g[(long long)sq * MR_NH + co];
      sb2 += hv > 0.f ? dq * cw3 : 0.f;
      sw3 += dq * hv;
      sb3 += dq;
    }
#pragma unroll
    for (int ks = 0; ks < MR_BC / 32; ++ks) {
      const bf16x8 d2a = *reinterpret_cast<const bf16x8*>(&sh.d2t[16 * w + r][32 * ks + 8 * g]);
      const bf16x8 d1a = *reinterpret_cast<const bf16x8*>(&sh.d1t[16 * w + r][32 * ks + 8 * g]);
#pragma unroll
      for (int nt = 0; nt < 4; ++nt)
        a2[nt] = mr_mfma(d2a, *reinterpret_cast<const bf16x8*>(&sh.h1t[16 * nt + r][32 * ks + 8 * g]), a2[nt]);
#pragma unroll
      for (int nt = 0; nt < MR_KP / 16; ++nt)
        a1[nt] = mr_mfma(d1a, *reinterpret_cast<const bf16x8*>(&sh.xt[16 * nt + r][32 * ks + 8 * g]), a1[nt]);
    }
  }
  float* G = part + (long long)blockIdx.x * MR_NPARAM;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int m = 16 * w + 4 * g + j;
#pragma unroll
    for (int nt = 0; nt < MR_KP / 16; ++nt) G[MR_OFF_W1 + m * MR_KP + 16 * nt + r] = a1[nt][j];
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) G[MR_OFF_W2 + m * MR_NH + 16 * nt + r] = a2[nt][j];
  }
#pragma unroll
  for (int nt = 0; nt < 4; ++nt) {
    sb1[nt] += __shfl_xor(sb1[nt], 16);
    sb1[nt] += __shfl_xor(sb1[nt], 32);
    if (g == 0) sh.red[0][w][16 * nt + r] = sb1[nt];
  }
  sh.red[1][w][co] = sb2;
  sh.red[2][w][co] = sw3;
  sh.red[3][w][co] = sb3;
  __syncthreads();
  const float v = sh.red[w][0][co] + sh.red[w][1][co] + sh.red[w][2][co] + sh.red[w][3][co];
  if (w == 0) G[MR_OFF_B1 + co] = v;
  else if (w == 1) G[MR_OFF_B2 + co] = v;
  else if (w == 2) G[MR_OFF_W3 + co] = v;
  else if (co < MR_NPARAM - MR_OFF_B3) G[MR_OFF_B3 + co] = co == 0 ? v : 0.f;   /* db3, then the padding */
}

/* G = the sum of n partial gradients, in order within four quarters */
__global__ __launch_bounds__(256) void k_grad_sum(int n, const float* part, float* G) {
  __shared__ float sh[4][64];
  const int e = blockIdx.x * 64 + threadIdx.x % 64, q = threadIdx.x / 64;
  const int p0 = n * q / 4, p1 = n * (q + 1) / 4;
  float a = 0.f;
  if (e < MR_NPARAM) {
#pragma unroll 8
    for (int p = p0; p < p1; ++p) a += part[(long long)p * MR_NPARAM + e];
  }
  sh[q][threadIdx.x % 64] = a;
  __syncthreads();
  if (q == 0 && e < MR_NPARAM) G[e] = (sh[0][threadIdx.x] + sh[1][threadIdx.x]) + (sh[2][threadIdx.x] + sh[3][threadIdx.x]);
}

/* Adam on the FP32 master parameters, refreshing the BF16 copy */
__global__ void k_adam(int n, float* w, __bf16* wb, const float* g, float* m, float* v, float lr, float b1,
                       float b2, float eps, float c1, float c2) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  const float gg = g[e];
  const float mm = b1 * m[e] + (1.f - b1) * gg;
  const float vv = b2 * v[e] + (1.f - b2) * gg * gg;
  m[e] = mm;
  v[e] = vv;
  const float ww = w[e] - lr * (mm / c1) / (sqrtf(vv / c2) + eps);
  w[e] = ww;
  wb[e] = (__bf16)ww;
}

/* activation cache of one batch and the partial gradients of its backward
   pass: one per work group of k_mlp_bwd, at most MR_NPART (a chunk of 64
   samples each up to 8192 samples) */
#define MR_NPART 128
static int mr_mlp_parts(int Bn) { return std::min((Bn + MR_BC - 1) / MR_BC, MR_NPART); }
struct mr_mlp_cache {
  float *h1, *h2, *z, *part;
  __bf16* h1b;
  size_t bytes;
};
static size_t mr_al(size_t x) { return (x + 255) & ~size_t(255); }
static mr_mlp_cache mr_mlp_cache_at(void* base, int Bn) {
  mr_mlp_cache C;
  char* p = (char*)base;
  size_t off = 0;
  auto take = [&](size_t bytes) { char* q = p ? p + off : nullptr; off += mr_al(bytes); return q; };
  const size_t B = (size_t)Bn;
  C.h1 = (float*)take(4 * B * MR_NH);
  C.h2 = (float*)take(4 * B * MR_NH);
  C.z = (float*)take(4 * B);
  C.h1b = (__bf16*)take(2 * B * MR_NH);
  C.part = (float*)take(4 * (size_t)mr_mlp_parts(Bn) * MR_NPARAM);
  C.bytes = off;
  return C;
}
/* whether the kernels may read x, params and the cache in 16-byte pieces */
static bool mr_mlp_aligned(const void* x, const void* params, const void* cache) {
  return (((uintptr_t)x | (uintptr_t)params | (uintptr_t)cache) & 15) == 0;
}

/* ------------------------------------------------------------ launchers */
extern "C" {

hipError_t mr_launch_fb_reset(hipStream_t s, int* cnt, int probe) {
  hipLaunchKernelGGL(k_fb_reset, dim3(1), dim3(64), 0, s, cnt, probe);
  return hipGetLastError();
}

hipError_t mr_launch_pack(hipStream_t s, const void* P, mr_learn_w* w) {
  const int n = MR_FRAG1 + MR_FRAG2 + MR_NH;
  hipLaunchKernelGGL(k_pack_weights, dim3((n + 255) / 256), dim3(256), 0, s, (const __bf16*)P, w);
  return hipGetLastError();
}

hipError_t mr_launch_learned(hipStream_t s, mr_inst* d, const mr_tile2* t, int nt, int stage, const mr_learn_w* w,
                             mr_band* band, int* cnt, int grid) {
  if (nt <= 0) return hipSuccess;
  const int G = grid > 0 && grid < nt ? grid : nt;
  hipLaunchKernelGGL(k2_learned, dim3(G), dim3(MR_BLOCK), 0, s, d, t, nt, stage, w, band, cnt);
  return hipGetLastError();
}

hipError_t mr_launch_fallback(hipStream_t s, mr_inst* d, const mr_band* band, int* cnt, int stage, int grid,
                              int any_bp) {
  hipLaunchKernelGGL(k_fb_direct<false>, dim3(grid), dim3(MR_BLOCK), 0, s, d, band, cnt, stage);
  if (any_bp) hipLaunchKernelGGL(k_fb_direct<true>, dim3(grid), dim3(MR_BLOCK), 0, s, d, band, cnt, stage);
  return hipGetLastError();
}

hipError_t mr_launch_features(hipStream_t s, const mr_inst* d, int inst, const int* cells, int n, void* out) {
  if (n <= 0) return hipSuccess;
  const long long tot = (long long)n * MR_KP;
  hipLaunchKernelGGL(k_features, dim3((unsigned)((tot + MR_BLOCK - 1) / MR_BLOCK)), dim3(MR_BLOCK), 0, s, d, inst,
                     cells, n, (__bf16*)out);
  return hipGetLastError();
}

size_t mr_mlp_cache_bytes(int batch) { return batch > 0 ? mr_mlp_cache_at(nullptr, batch).bytes : 0; }

hipError_t mr_mlp_gemm(hipStream_t s, int M, int N, int K, const void* A, long long sAm, long long sAk,
                       const void* B, long long sBk, long long sBn, void* C, long long sCm, long long sCn) {
  const int tiles = ((M + 15) / 16) * ((N + 15) / 16);
  hipLaunchKernelGGL(k_gemm_bf16, dim3((tiles + 3) / 4), dim3(MR_BLOCK), 0, s, M, N, K, (const __bf16*)A, sAm, sAk,
                     (const __bf16*)B, sBk, sBn, (float*)C, sCm, sCn);
  return hipGetLastError();
}

hipError_t mr_mlp_forward(hipStream_t s, const void* x, const void* params, void* cache, void* z, int Bn) {
  const mr_mlp_cache C = mr_mlp_cache_at(cache, Bn);
  const auto k = mr_mlp_aligned(x, params, cache) ? k_mlp_fwd<true> : k_mlp_fwd<false>;
  hipLaunchKernelGGL(k, dim3((Bn + 15) / 16), dim3(64), 0, s, Bn, (const __bf16*)x, (const __bf16*)params, C.h1, C.h1b,
                     C.h2, C.z, (float*)z);
  return hipGetLastError();
}

hipError_t mr_mlp_backward(hipStream_t s, const void* x, const void* params, void* cache, const void* labels,
                           void* grads, void* loss, int Bn) {
  const mr_mlp_cache C = mr_mlp_cache_at(cache, Bn);
  const int n = mr_mlp_parts(Bn);
  const auto k = mr_mlp_aligned(x, params, cache) ? k_mlp_bwd<true> : k_mlp_bwd<false>;
  hipLaunchKernelGGL(k, dim3(n), dim3(256), 0, s, Bn, (const __bf16*)x, (const __bf16*)params, C.z,
                     (const float*)labels, C.h1, C.h1b, C.h2, (float*)loss, C.part);
  hipLaunchKernelGGL(k_grad_sum, dim3((MR_NPARAM + 63) / 64), dim3(256), 0, s, n, C.part, (float*)grads);
  return hipGetLastError();
}

hipError_t mr_mlp_adam(hipStream_t s, void* master, void* params, const void* grads, void* m, void* v, int step,
                       float lr, float beta1, float beta2, float eps) {
  const float c1 = 1.f - powf(beta1, (float)step), c2 = 1.f - powf(beta2, (float)step);
  hipLaunchKernelGGL(k_adam, dim3((MR_NPARAM + 255) / 256), dim3(256), 0, s, MR_NPARAM, (float*)master,
                     (__bf16*)params, (const float*)grads, (float*)m, (float*)v, lr, beta1, beta2, eps, c1, c2);
  return hipGetLastError();
}

}  /* extern "C" */
