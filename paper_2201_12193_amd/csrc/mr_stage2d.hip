/* The 2D stage kernel (its own translation unit: it keeps the constant
 * table of the reconstruction in LDS, see mr_device.h, and is compiled
 * with its own scheduling options, see build.py). */
#define MR_KT_IN_LDS 1
#include "mr_common.h"

/* 2D stage kernel.  A work group owns a strip of CW = 256/NC consecutive
 * cells in x (two of them ring cells) and sweeps it upward over `rows` rows
 * plus one ring row below and one above.
 *
 * Moments (the strip plus two columns each side) sit in LDS rings: the cell
 * averages and y moments of rows y-2..y+2 (five rows: the modification of
 * the stencil's upper and lower cells reads rows y +- 2), the x moments of
 * rows y-1..y+1 (three rows); each value is loaded from HBM once per work
 * group, with the boundary condition applied when it is stored, and the
 * rows needed next are fetched into registers while the current row is
 * computed.  Flags of rows y-1..y+1 sit in a three-row LDS ring.
 *
 * Stage 1 also writes the first moments of U^n after Step 2.2 (I.unm), which
 * the combination of stages 2 and 3 uses.
 *
 * With NC = 4 a wave holds 16 cells, lane = 16 k + cell: the four lanes of a
 * cell each reconstruct one conserved component, then each lane takes one
 * row eta_r of the cell's 4x4 Gauss-Lobatto grid for the volume integrals,
 * the left-face flux at eta_r and the bottom-face flux at xi_r.  The sums
 * over the rows and points, with their quadrature weights, are 4x4x4 FP64
 * matrix products (mr2_sum): the contraction index of that instruction is
 * lane / 16, so the lanes' values are its operand as they stand.  The
 * top-face flux of a row is the bottom-face flux of the next one, so the
 * residual of row j is completed while row j+1 is processed; the row's top
 * trace waits in registers.  mode 0..2 = RK stage, 3 = write L(U).
 *
 * CH (characteristic-wise Step 1, NC = 4): lane k reconstructs field k of
 * the x set into the value slots, maps row eta_k of the cell back to the
 * conserved variables (R), takes the x-flux volume integral of that row
 * and the left-face flux; then the same with the y set for the y-flux
 * volume integral and the bottom-face flux.  The moment rows of the next
 * step are stored once both sets have read the stencil.
 *
 * What bounds it: FP64 issue, two thirds of the issue slots at the 2.1 GHz
 * the clock holds under this load; the rest are waits of the two waves a SIMD
 * for LDS and at barriers.  By the counters a wave takes 945 vector
 * instructions a row step, 740 of them FP64 and 15 FP64 matrix products
 * (1,300 and 900 before the factored basis of Step 1, the one-sided HLLC, the
 * sums as matrix products, the top trace in registers and the ghost rules
 * out of the staging of strips without ghosts), two waves a SIMD at 228
 * VGPRs and 76 KB of LDS a work group.  2048 x 2048, 56-row strips on 512
 * work groups: 983 -> 788 us a launch (31 TFLOP/s of the 71.8 an FP64 matrix
 * product reaches); 800 x 200 with inflow sides, 8-row strips: 109 -> 101;
 * 600 x 200 characteristic-wise: 254 -> 235.  Strips of 128 or 64 threads
 * (30 or 14 owned columns) took 1.3 times as long: their narrower ring
 * costs more than the shorter barriers give. */
template <int NC>
struct mr2_lds {
  static constexpr int CW = MR_BLOCK / NC;   /* strip cells incl. ring */
  static constexpr int XW = CW + 4;          /* staged columns */
  static constexpr int NP = 3 * NC;          /* staged planes per row step */
  /* strides (in doubles) that put the two groups of 16 cells a half wave
     accesses 16 doubles apart modulo the 32 the banks hold; val reaches the
     same with an exchange of 16-cell groups in the odd components */
  static constexpr int CS = CW;              /* component stride of val */
  static constexpr int VS = NC * CS + 4;     /* point stride of val */
  static constexpr int FC = CW + 16;         /* component stride of fs */
  static constexpr int FS = NC * FC + 16;    /* quantity stride of fs */
  static constexpr int XP = NC == 1 ? XW : CW + 8;    /* plane stride of mA */
  static constexpr int XB = NC == 1 ? XW : CW + 16;   /* plane stride of mB */
  double mA[5][2 * NC][XP];   /* planes (c, m = 0) and (c, m = 2): index 2c, 2c+1 */
  double mB[3][NC][XB];       /* planes (c, m = 1)                               */
  unsigned char flg[3][XW];
  double val[16 * VS];
  double fs[4 * FS];          /* left-face sums (weights w, w eta), bottom-face sums */
};

/* The sum over the four lanes of a cell of b times the A operand's weights
   (a: the weight of the lane's row, lane 16 k + cell), the same in every lane
   of the cell: an operand of equal rows, so that the sum of one component,
   should it not be finite, stays in that component (weights that are zero in
   the other rows would hand a NaN on to them). */
MR_INL double mr2_sum(double a, double b) {
#ifdef __HIP_DEVICE_COMPILE__
  return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, 0.0, 0, 0, 0);
#else
  return a * b;
#endif
}
/* component k of four values */
MR_INL double mr2_pick(int k, const double v[4]) {
  const double a = k == 1 ? v[1] : v[0], b = k == 3 ? v[3] : v[2];
  return k < 2 ? a : b;
}

MR_INL int mr_mod3(int y) { return ((y % 3) + 3) % 3; }
MR_INL int mr_mod5(int y) { return ((y % 5) + 5) % 5; }

/* staged element e of a row step at row y (A planes at row y+1, B planes
   at row y): plane pl < 2 NC is A plane pl, else B plane pl - 2 NC */
template <int NC, int XW, bool STEP>
MR_INL double mr2_stage_ld(const mr_grid& g, int e, int xs0, int y) {
  const int pl = e / XW, col = e % XW;
  if (pl < 2 * NC) return mr_ld<STEP>(g, pl / 2, (pl % 2) * 2, xs0 + col, y + 1);
  return mr_ld<STEP>(g, pl - 2 * NC, 1, xs0 + col, y);
}

/* the eigenvectors of direction D at the cell of staged column c0 whose row
   sits in slot r; taken afresh where they are needed again (holding them
   through Step 1 spills) */
template <int D>
MR_INL mr_char2 mr2_stage_char(const mr2_lds<4>& sh, int r, int c0, double gam) {
  double u0[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) u0[c] = sh.mA[r][2 * c][c0];
  return mr_char2_state<D>(u0, gam);
}

/* Characteristic-wise Step 1 (see mr_char2): field k of direction D of the
   cell at staged column c0, projected from the stencil in the LDS rings
   (the troubled cells' first moments modified when the cell is troubled)
   and reconstructed. */
template <bool BP, int D>
MR_INL void mr2_stage_field(const mr2_lds<4>& sh, const int* ra, const int* rb, const int* fs, int c0, int k,
                            double gam, const mr_wconst& W, double val[16]) {
  double lk[4];
  mr_char2_left<D>(mr2_stage_char<D>(sh, ra[2], c0, gam), k, lk);
  double u[9], v[9], w[9];
#pragma unroll
  for (int dy = 0; dy < 3; ++dy)
#pragma unroll
    for (int dx = 0; dx < 3; ++dx) {
      const int l = dx + 3 * dy, cc = c0 + dx - 1;
      double a = 0.0, b = 0.0, d = 0.0;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        a += lk[c] * sh.mA[ra[dy + 1]][2 * c][cc];
        b += lk[c] * sh.mB[rb[dy]][c][cc];
        d += lk[c] * sh.mA[ra[dy + 1]][2 * c + 1][cc];
      }
      u[l] = a; v[l] = b; w[l] = d;
    }
  if (fs[4]) {
#pragma unroll
    for (int dy = 0; dy < 3; ++dy)
#pragma unroll
      for (int dx = 0; dx < 3; ++dx) {
        const int l = dx + 3 * dy, cc = c0 + dx - 1;
        if (!fs[l]) continue;
        double b = 0.0, d = 0.0;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          b += lk[c] * mr_modified_moment(sh.mA[ra[dy + 1]][2 * c][cc - 1], sh.mA[ra[dy + 1]][2 * c][cc + 1],
                                          sh.mB[rb[dy]][c][cc - 1], sh.mB[rb[dy]][c][cc + 1]);
          d += lk[c] * mr_modified_moment(sh.mA[ra[dy]][2 * c][cc], sh.mA[ra[dy + 2]][2 * c][cc],
                                          sh.mA[ra[dy]][2 * c + 1][cc], sh.mA[ra[dy + 2]][2 * c + 1][cc]);
        }
        v[l] = b; w[l] = d;
      }
  }
  mr_recon2d<BP>(u, v, w, W, val);
}

template <int NC, bool BP, int GB, bool CH>
__global__ __launch_bounds__(MR_BLOCK) MR_OCC void k2_stage(const mr_inst* __restrict__ insts, const mr_tile2* __restrict__ tiles, int ntiles, int mode) {
  mr_kt_fill();
  using S = mr2_lds<NC>;
  constexpr int CW = S::CW, XW = S::XW, NP = S::NP, CS = S::CS, VS = S::VS, FC = S::FC, FS = S::FS;
  __shared__ S sh;
  const int tid = threadIdx.x;
  const int k = (NC == 1) ? 0 : (tid >> 4) & 3;
  const int cs = (NC == 1) ? tid : 16 * (tid >> 6) + (tid & 15);
  const int comp = k;
#define VAL(p, c, cell) sh.val[(p) * VS + (c) * CS + ((cell) ^ (NC == 1 ? 0 : ((c) & 1) << 4))]
#define FSM(m, c, cell) sh.fs[(m) * FS + (c) * FC + (cell)]
  /* staging: thread (component gc, column tid % CW) loads its column's three
     moments in every row step; the four columns beyond CW are the first 12
     threads' of each component (moment em, column ecol).  The moments are
     staged at different rows (x moments one row behind) */
  const int gc = NC == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid / CW);
  const int gcol = tid % CW, em = gcol >> 2, ecol = CW + (gcol & 3);
  const bool ext = gcol < 12;
  /* quadrature weights of this lane's row as A operands (see mr2_sum): the
     volume sums, and in alternate output rows the face sums with weights w
     and w eta */
  const double aF = glw(k) * MR_W0, aS = (tid & 1) ? glw(k) * gln(k) : glw(k);
  for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
    const mr_tile2 tl = tiles[t];
    const mr_inst& I = insts[tl.inst];
    if (mode < 3 && !I.active) continue;
    const int st = mode == 3 ? 0 : mode;
    const mr_grid g{mr_gp(I.p_in[st]), I.plane, I.nx, I.ny, I.bcx, I.bcy, 3, GB ? &I : nullptr, mr_stage_time(I, mode)};
    const mr_grid gn{mr_gp(I.p_un), I.plane, I.nx, I.ny, I.bcx, I.bcy, 3, GB ? &I : nullptr, mr_stage_time(I, 0)};
    const MR_GLB unsigned char* fl = mr_gp(I.flags[(mode == 0 || mode == 3) ? 0 : 1]);
    MR_GLB double* unm = mr_gp(I.unm);
    const double rdx = I.rdx, rdy = I.rdy, dt = I.dt, gam = I.gam;
    const double alpha = (NC == 1) ? mr_bitsd(I.lfa[st]) : 0.0;
    MR_GLB double* O = mr_gp(I.p_out[st]);
    const long long P = I.plane;
    const int nx = I.nx;
    const int xs0 = tl.x0 - 3;                 /* strip column 0 */
    const int x = tl.x0 - 1 + cs;
    const bool outx = cs >= 1 && cs <= CW - 2 && x < I.nx;
    /* folded columns of this thread's staged elements and their x ghost
       kinds; xplain: no staged column of the strip is a ghost that changes
       its value (uniform) */
    int kx = 0, kxe = 0;
    const int ii = mr_fold(xs0 + gcol, nx, I.bcx, &kx);
    const int iie = mr_fold(xs0 + ecol, nx, I.bcx, &kxe);
    const bool xplain = (xs0 >= 0 || (I.bcx & 3) == 0) && (xs0 + XW <= nx || ((I.bcx >> 2) & 3) == 0);
    const MR_GLB double* ub = g.U + (long long)(3 * gc) * P;      /* component gc */
    const MR_GLB double* ue = ub + (ext ? (long long)em * P + iie : 0);
    /* value of a staged element of moment m: zero as a first moment of a
       transmissive ghost, the sign of a reflective one */
    auto ghost = [&](double v, int m, int kxx, int ky) {
      const bool neg = (kxx == 2 && mr_refl_flip(gc, m, 0)) != (ky == 2 && mr_refl_flip(gc, m, 1));
      return (m != 0 && (kxx == 1 || ky == 1)) ? 0.0 : (neg ? -v : v);
    };
    auto flag_ld = [&](int e, int row) { return (unsigned char)mr_flag(fl, I.fex, I.fey, I.fhalo, xs0 + e, row); };
    /* ---- prologue: A rows y0-3 .. y0+1, B and flag rows y0-2 .. y0 ---- */
    for (int r = tl.y0 - 3; r <= tl.y0 - 2; ++r)
      for (int e = tid; e < 2 * NC * XW; e += MR_BLOCK)
        sh.mA[mr_mod5(r)][e / XW][e % XW] = mr_ld<GB == 2>(g, (e / XW) / 2, ((e / XW) % 2) * 2, xs0 + e % XW, r);
    for (int r = tl.y0 - 2; r <= tl.y0; ++r) {
      for (int e = tid; e < NP * XW; e += MR_BLOCK) {
        const double v = mr2_stage_ld<NC, XW, GB == 2>(g, e, xs0, r);
        if (e / XW < 2 * NC) sh.mA[mr_mod5(r + 1)][e / XW][e % XW] = v;
        else sh.mB[mr_mod3(r)][e / XW - 2 * NC][e % XW] = v;
      }
      for (int e = tid; e < XW; e += MR_BLOCK) sh.flg[mr_mod3(r)][e] = flag_ld(e, r);
    }
    __syncthreads();
    double pAu = 0.0, pAv = 0.0, pAw = 0.0, pU = 0.0, pV = 0.0, pW = 0.0;
    double tp[4 / NC][NC];   /* top trace of the row below at this lane's points */
#pragma unroll
    for (int rr = 0; rr < 4 / NC; ++rr)
#pragma unroll
      for (int c = 0; c < NC; ++c) tp[rr][c] = 0.0;
    for (int jr = -1; jr <= tl.rows; ++jr) {
      const int y = tl.y0 + jr;
      /* stages 2 and 3: U^n of the row finished in this step, loaded now so
         that the latency hides behind the reconstruction */
      double qun = 0.0, qvn = 0.0, qwn = 0.0;
      if ((mode == 1 || mode == 2) && jr >= 1 && outx) {
        const long long cell = (long long)(y - 1) * nx + x;
        const MR_GLB double* vs = I.mod == 0 ? unm + (long long)(comp * 2) * P : gn.U + (long long)(comp * 3 + 1) * P;
        qun = gn.U[(long long)(comp * 3) * P + cell];
        qvn = vs[cell];
        qwn = vs[P + cell];
      }
      /* prefetch A row y+3, B and flag row y+2 (stored once rows y-2 and
         y-1 are consumed); the row folds are uniform over the work group */
      int kA = 0, kB = 0;
      const long long jA = (long long)mr_fold(y + 3, I.ny, I.bcy, &kA) * nx;
      const long long jB = (long long)mr_fold(y + 2, I.ny, I.bcy, &kB) * nx;
      const double pre0 = (ub + jA)[ii], pre1 = (ub + P + jB)[ii], pre2 = (ub + 2 * P + jA)[ii];
      double pree = 0.0;
      if (ext) pree = ue[em == 1 ? jB : jA];
      unsigned char pref = 0, prefe = 0;
      if (tid < XW) pref = flag_ld(tid, y + 2);
      if (XW > MR_BLOCK && tid < XW - MR_BLOCK) prefe = flag_ld(MR_BLOCK + tid, y + 2);
      /* ---- Steps 1, 2.2, 2.3 for component `comp` of cell (x, y) ---- */
      double cu = 0.0, cv = 0.0, cw = 0.0;
      /* characteristic-wise: the stencil rows, flags and the cell's state */
      int cra[5], crb[3], cfs[9];
      if constexpr (CH) {
        const int c0 = cs + 2;
        for (int q = 0; q < 5; ++q) cra[q] = mr_mod5(y - 2 + q);
        for (int q = 0; q < 3; ++q) crb[q] = mr_mod3(y - 1 + q);
#pragma unroll
        for (int l = 0; l < 9; ++l) cfs[l] = sh.flg[crb[l / 3]][c0 + l % 3 - 1];
          /* the cell's own moments for the combination */
          const bool md = cfs[4] && I.mod != 1;
          cu = sh.mA[cra[2]][2 * comp][c0];
          cv = md ? mr_modified_moment(sh.mA[cra[2]][2 * comp][c0 - 1], sh.mA[cra[2]][2 * comp][c0 + 1],
                                       sh.mB[crb[1]][comp][c0 - 1], sh.mB[crb[1]][comp][c0 + 1])
                  : sh.mB[crb[1]][comp][c0];
          cw = md ? mr_modified_moment(sh.mA[cra[1]][2 * comp][c0], sh.mA[cra[3]][2 * comp][c0],
                                       sh.mA[cra[1]][2 * comp + 1][c0], sh.mA[cra[3]][2 * comp + 1][c0])
                  : sh.mA[cra[2]][2 * comp + 1][c0];
        double val[16];
        mr2_stage_field<BP, 0>(sh, cra, crb, cfs, c0, comp, gam, I.W, val);
#pragma unroll
        for (int q = 0; q < 16; ++q) VAL(q, comp, cs) = val[q];
      } else {
        const int ra[5] = {mr_mod5(y - 2), mr_mod5(y - 1), mr_mod5(y), mr_mod5(y + 1), mr_mod5(y + 2)};
        const int rb[3] = {mr_mod3(y - 1), mr_mod3(y), mr_mod3(y + 1)};
        const int c0 = cs + 2;                    /* staged column of cell x */
        double u[9], v[9], w[9];
        int fs[9];
#pragma unroll
        for (int dy = 0; dy < 3; ++dy)
#pragma unroll
          for (int dx = 0; dx < 3; ++dx) {
            const int l = dx + 3 * dy;
            u[l] = sh.mA[ra[dy + 1]][2 * comp][c0 + dx - 1];
            v[l] = sh.mB[rb[dy]][comp][c0 + dx - 1];
            w[l] = sh.mA[ra[dy + 1]][2 * comp + 1][c0 + dx - 1];
          }
        fs[4] = sh.flg[rb[1]][c0];
        if (fs[4]) {
          /* troubled cell: first moments of the troubled cells of the
             stencil modified from the unmodified input (Jacobi) */
#pragma unroll
          for (int dy = 0; dy < 3; ++dy)
#pragma unroll
            for (int dx = 0; dx < 3; ++dx) {
              const int l = dx + 3 * dy;
              fs[l] = sh.flg[rb[dy]][c0 + dx - 1];
              if (!fs[l]) continue;
              const int cc = c0 + dx - 1;
              v[l] = mr_modified_moment(sh.mA[ra[dy + 1]][2 * comp][cc - 1], sh.mA[ra[dy + 1]][2 * comp][cc + 1],
                                        sh.mB[rb[dy]][comp][cc - 1], sh.mB[rb[dy]][comp][cc + 1]);
              w[l] = mr_modified_moment(sh.mA[ra[dy]][2 * comp][cc], sh.mA[ra[dy + 2]][2 * comp][cc],
                                        sh.mA[ra[dy]][2 * comp + 1][cc], sh.mA[ra[dy + 2]][2 * comp + 1][cc]);
            }
        }
        cu = u[4];
        /* the combination takes the modified first moments unless the
           modification stays internal to L */
        cv = I.mod == 1 ? sh.mB[rb[1]][comp][c0] : v[4];
        cw = I.mod == 1 ? sh.mA[ra[2]][2 * comp + 1][c0] : w[4];
        double val[16];
        mr_recon2d<BP>(u, v, w, I.W, val);
#pragma unroll
        for (int q = 0; q < 16; ++q) VAL(q, comp, cs) = val[q];
      }
      __syncthreads();
      /* the slots of A row y-2 and of B/flag row y-1 are consumed: store
         A row y+3 and B/flag row y+2 */
      auto store_rows = [&]() {
        const int sa = mr_mod5(y + 3), sb = mr_mod3(y + 2);
        if (xplain && kA == 0 && kB == 0) {
          sh.mA[sa][2 * gc][gcol] = pre0;
          sh.mB[sb][gc][gcol] = pre1;
          sh.mA[sa][2 * gc + 1][gcol] = pre2;
          if (ext) (em == 1 ? sh.mB[sb][gc] : sh.mA[sa][2 * gc + (em >> 1)])[ecol] = pree;
        } else {
          sh.mA[sa][2 * gc][gcol] = ghost(pre0, 0, kx, kA);
          sh.mB[sb][gc][gcol] = ghost(pre1, 1, kx, kB);
          sh.mA[sa][2 * gc + 1][gcol] = ghost(pre2, 2, kx, kA);
          if (ext)
            (em == 1 ? sh.mB[sb][gc] : sh.mA[sa][2 * gc + (em >> 1)])[ecol] = ghost(pree, em, kxe, em == 1 ? kB : kA);
        }
        if (tid < XW) sh.flg[sb][tid] = pref;
        if (XW > MR_BLOCK && tid < XW - MR_BLOCK) sh.flg[sb][MR_BLOCK + tid] = prefe;
        if (GB && mr_presc_rows<GB == 2>(I, xs0, XW, y + 2, 2)) {
          /* ghosts that hold prescribed data, by the threads that stored them */
          const double tb = mr_stage_time(I, mode);
#pragma unroll 1
          for (int q = 0; q < 4; ++q) {
            if (q == 3 && !ext) continue;
            const int m = q < 3 ? q : em, col = q < 3 ? gcol : ecol, row = m == 1 ? y + 2 : y + 3;
            double v;
            if (mr_presc(I, gc, m, xs0 + col, row, tb, &v) ||
                (GB == 2 && mr_step_val(I, g.U, gc, m, xs0 + col, row, &v))) {
              if (m == 1) sh.mB[sb][gc][col] = v;
              else sh.mA[sa][2 * gc + (m >> 1)][col] = v;
            }
          }
        }
      };
      /* ---- volume integrals and the fluxes this lane owns ---- */
      /* F, G: twelve times the xi quadrature of the row; fx, gy: the fluxes */
      double F[4 / NC][NC], G[4 / NC][NC], fx[4 / NC][NC], gy[4 / NC][NC];
#pragma unroll
      for (int rr = 0; rr < 4 / NC; ++rr)
#pragma unroll
        for (int c = 0; c < NC; ++c) F[rr][c] = G[rr][c] = fx[rr][c] = gy[rr][c] = 0.0;
      double fF = 0.0, fG = 0.0;
      const bool body = jr >= 0 && jr < tl.rows;
      if constexpr (CH) {
        /* lane k = row eta_k of the cell: x set back to conserved variables */
        const int r = k;
        double pts[4][4], fq[4][4];
        mr_char2 ec = mr2_stage_char<0>(sh, cra[2], cs + 2, gam);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          double wq[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) wq[j] = VAL(q + 4 * r, j, cs);
          mr_char2_right<0>(ec, wq, pts[q]);
        }
        /* row eta_k of the cell is read and written by lane k only */
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int c = 0; c < 4; ++c) VAL(q + 4 * r, c, cs) = pts[q][c];
        if (body) {
#pragma unroll
          for (int q = 0; q < 4; ++q) mr_euler_flux<4, 0>(pts[q], gam, fq[q]);
#pragma unroll
          for (int c = 0; c < 4; ++c) F[0][c] = (fq[0][c] + fq[3][c]) + 5.0 * (fq[1][c] + fq[2][c]);
        }
        __syncthreads();
        if (body && cs >= 1) {
          double a[4];
#pragma unroll
          for (int c = 0; c < 4; ++c) a[c] = VAL(3 + 4 * r, c, cs - 1);
          mr_face_flux<4, 0, GB == 2>(I, a, pts[0], gam, alpha, x, y, mr_stage_time(I, mode), fx[0]);
        }
        __syncthreads();
        /* the x set's sums at once, the face sums straight to LDS: one value
           instead of eight held through the y set's Step 1 */
        {
          double sF[4], sx[4];
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            sF[c] = mr2_sum(aF, F[0][c]);
            sx[c] = mr2_sum(aS, fx[0][c]);
          }
          fF = mr2_pick(k, sF);
          if (k < 2) {
#pragma unroll
            for (int c = 0; c < 4; ++c) FSM(k, c, cs) = sx[c];
          }
        }
        /* field k of the y set (the stencil rows are still in place) */
        {
          const int c0 = cs + 2;
          double val[16];
          mr2_stage_field<BP, 1>(sh, cra, crb, cfs, c0, comp, gam, I.W, val);
#pragma unroll
          for (int q = 0; q < 16; ++q) VAL(q, comp, cs) = val[q];
        }
        __syncthreads();
        store_rows();
        ec = mr2_stage_char<1>(sh, cra[2], cs + 2, gam);   /* row y's slot is not the one stored */
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          double wq[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) wq[j] = VAL(q + 4 * r, j, cs);
          mr_char2_right<1>(ec, wq, pts[q]);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int c = 0; c < 4; ++c) VAL(q + 4 * r, c, cs) = pts[q][c];
        if (body) {
#pragma unroll
          for (int q = 0; q < 4; ++q) mr_euler_flux<4, 1>(pts[q], gam, fq[q]);
#pragma unroll
          for (int c = 0; c < 4; ++c) G[0][c] = (fq[0][c] + fq[3][c]) + 5.0 * (fq[1][c] + fq[2][c]);
        }
        __syncthreads();
        if (jr >= 0) {
          double b[4];
#pragma unroll
          for (int c = 0; c < 4; ++c) b[c] = VAL(r, c, cs);
          mr_face_flux<4, 1, GB == 2>(I, tp[0], b, gam, alpha, y, x, mr_stage_time(I, mode), gy[0]);
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) tp[0][c] = VAL(12 + r, c, cs);
      } else {
        store_rows();
#pragma unroll
        for (int rr = 0; rr < 4 / NC; ++rr) {
          const int r = (NC == 1) ? rr : k;
          if (body) {
            double pts[4][NC], f[4][NC], gg[4][NC];
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
              for (int c = 0; c < NC; ++c) pts[q][c] = VAL(q + 4 * r, c, cs);
            if constexpr (NC == 4) {
              double rr4[4];
              mr_recip4(pts[0][0], pts[1][0], pts[2][0], pts[3][0], rr4);
#pragma unroll
              for (int q = 0; q < 4; ++q) mr_euler_fg_r(pts[q], rr4[q], gam, f[q], gg[q]);
            } else {
#pragma unroll
              for (int q = 0; q < 4; ++q) f[q][0] = gg[q][0] = 0.5 * pts[q][0] * pts[q][0];
            }
#pragma unroll
            for (int c = 0; c < NC; ++c) F[rr][c] = (f[0][c] + f[3][c]) + 5.0 * (f[1][c] + f[2][c]);
#pragma unroll
            for (int c = 0; c < NC; ++c)
              G[rr][c] = (NC == 4 && c == 1) ? F[rr][NC / 2] : (gg[0][c] + gg[3][c]) + 5.0 * (gg[1][c] + gg[2][c]);
            if (cs >= 1) {
              double a[NC];
#pragma unroll
              for (int c = 0; c < NC; ++c) a[c] = VAL(3 + 4 * r, c, cs - 1);
              mr_face_flux<NC, 0, GB == 2>(I, a, pts[0], gam, alpha, x, y, mr_stage_time(I, mode), fx[rr]);
            }
          }
          if (jr >= 0) {
            double b[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) b[c] = VAL(r, c, cs);
            mr_face_flux<NC, 1, GB == 2>(I, tp[rr], b, gam, alpha, y, x, mr_stage_time(I, mode), gy[rr]);
          }
#pragma unroll
          for (int c = 0; c < NC; ++c) tp[rr][c] = VAL(12 + r, c, cs);
        }
      }
      /* the quadratures over the rows: lane k receives component k's volume
         sums; the face sums of all components go through LDS */
      if constexpr (NC == 4) {
        /* face sums: rows 0, 1 (lanes 0, 1 of a cell) the left face's, which
           CH has written, 2, 3 the bottom face's */
        double sF[4], sG[4], sy[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          if (!CH) sF[c] = mr2_sum(aF, F[0][c]);
          sG[c] = mr2_sum(aF, G[0][c]);
          const double sx = CH ? 0.0 : mr2_sum(aS, fx[0][c]);
          sy[c] = mr2_sum(aS, gy[0][c]);
          if (!CH) FSM(k, c, cs) = k < 2 ? sx : sy[c];
        }
        if (CH && k >= 2) {
#pragma unroll
          for (int c = 0; c < 4; ++c) FSM(k, c, cs) = sy[c];
        }
        if (!CH) fF = mr2_pick(k, sF);
        fG = mr2_pick(k, sG);
      } else {
        double q0 = 0.0, q1 = 0.0, q2 = 0.0, q3 = 0.0;
#pragma unroll
        for (int rr = 0; rr < 4 / NC; ++rr) {
          const double wr = glw(rr), we = glw(rr) * gln(rr);
          fF += wr * MR_W0 * F[rr][0]; fG += wr * MR_W0 * G[rr][0];
          q0 += wr * fx[rr][0]; q1 += we * fx[rr][0];
          q2 += wr * gy[rr][0]; q3 += we * gy[rr][0];
        }
        FSM(0, 0, cs) = q0; FSM(1, 0, cs) = q1; FSM(2, 0, cs) = q2; FSM(3, 0, cs) = q3;
      }
      /* (the next row's values are written after this barrier, its face sums
         after the one that follows, so the row needs no third) */
      __syncthreads();
      const double xl0 = FSM(0, comp, cs), xl1 = FSM(1, comp, cs);
      const double yb0 = FSM(2, comp, cs), yb1 = FSM(3, comp, cs);
      const int cr = cs + 1 < CW ? cs + 1 : cs;
      const double xr0 = FSM(0, comp, cr), xr1 = FSM(1, comp, cr);
      /* ---- finish the row below: its top face is this row's bottom face ---- */
      if (jr >= 1 && outx) {
        const int yp = y - 1;
        const double Lu = pAu - yb0 * rdy;
        const double Lv = pAv - yb1 * rdy;
        const double Lw = pAw - yb0 * (0.5 * rdy);
        double r0, r1, r2;
        const long long cell = (long long)yp * nx + x;
        if (mode == 3) { r0 = Lu; r1 = Lv; r2 = Lw; }
        else if (mode == 0) {
          r0 = pU + dt * Lu; r1 = pV + dt * Lv; r2 = pW + dt * Lw;
          /* U^n after Step 2.2 (its first moments) for stages 2 and 3 */
          if (I.mod == 0) {
            const bool sol = GB == 2 && mr_solid(I, x, yp);
            unm[(long long)(comp * 2 + 0) * P + cell] = sol ? 0.0 : pV;
            unm[(long long)(comp * 2 + 1) * P + cell] = sol ? 0.0 : pW;
          }
        } else {
          const double a = mode == 1 ? 0.75 : 1.0 / 3.0, b = mode == 1 ? 0.25 : 2.0 / 3.0;
          const double un = qun, vn = qvn, wn = qwn;
          r0 = a * un + b * pU + b * dt * Lu;
          r1 = a * vn + b * pV + b * dt * Lv;
          r2 = a * wn + b * pW + b * dt * Lw;
        }
        if (GB == 2 && mr_solid(I, x, yp)) r0 = r1 = r2 = 0.0;   /* the step's cells carry no state */
        O[(long long)(comp * 3 + 0) * P + cell] = r0;
        O[(long long)(comp * 3 + 1) * P + cell] = r1;
        O[(long long)(comp * 3 + 2) * P + cell] = r2;
      }
      /* ---- this row's partial residual (all but the top face) ---- */
      pAu = -(xr0 - xl0) * rdx + yb0 * rdy;
      pAv = (fF - 0.5 * (xr0 + xl0)) * rdx + yb1 * rdy;
      pAw = (fG - 0.5 * yb0) * rdy - (xr1 - xl1) * rdx;
      pU = cu;
      pV = cv;
      pW = cw;
    }
  }
#undef VAL
#undef FSM
}

/* gb: 0 no instance of the list has per-side boundary data (the variant
   without that code), 1 some have ghosts that hold a prescribed state, 2
   some also have a step or the wall flux (Euler); ch: the
   characteristic-wise Step 1 (nc = 4) */
extern "C" hipError_t mr_launch_stage2(hipStream_t s, int nc, int bp, int gb, int ch, mr_inst* d, const mr_tile2* t,
                                       int nt, int mode, int grid) {
  if (nt <= 0) return hipSuccess;
  const dim3 G(grid > 0 && grid < nt ? grid : nt), B(MR_BLOCK);
#define MR_L2(NC_, BP_, CH_)                                                                           \
  do {                                                                                                 \
    if (gb == 2 && NC_ == 4) hipLaunchKernelGGL((k2_stage<NC_, BP_, 2, CH_>), G, B, 0, s, d, t, nt, mode); \
    else if (gb) hipLaunchKernelGGL((k2_stage<NC_, BP_, 1, CH_>), G, B, 0, s, d, t, nt, mode);         \
    else hipLaunchKernelGGL((k2_stage<NC_, BP_, 0, CH_>), G, B, 0, s, d, t, nt, mode);                 \
  } while (0)
  if (nc == 1) { if (bp) MR_L2(1, true, false); else MR_L2(1, false, false); }
  else if (nc == 4 && !ch) { if (bp) MR_L2(4, true, false); else MR_L2(4, false, false); }
  else if (nc == 4) { if (bp) MR_L2(4, true, true); else MR_L2(4, false, true); }
  else return hipErrorInvalidValue;
#undef MR_L2
  return hipGetLastError();
}
