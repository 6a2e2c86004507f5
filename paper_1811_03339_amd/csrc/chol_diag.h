// Factorization of one 64 x 64 diagonal block of the blocked Cholesky in
// LDS (256 threads), shared by the first-panel kernel and the trailing
// updates whose tile (0, 0) factors the next diagonal block.
#pragma once

#include "dense.h"

namespace fpde {

// LDS used by one diagonal-block factorization: the block on entry (lower
// part, zeros above; identity past the matrix end); on exit L in the lower
// triangle and Z = inv(L)^T in the strict upper triangle, Z's diagonal in dinv.
struct DiagSmem {
  double L[NB][NB + 1];
  double dinv[NB];
};

// Factor the 64 x 64 diagonal block held in sm.L (rows/columns >= nb are
// identity), write L over A's block at (k0, k0), inv(L) to Linv and
// inv(L)^T to LinvT.  The first 256 threads of the workgroup work; further
// threads only take part in its barriers.
//
// What bounds it is the dependent chain of 64 pivots, so everything is
// arranged around that chain.  The column operations that turn the block
// into L turn the identity below it into Z = inv(L)^T, so the two are
// factored together as one tall matrix in 16-column panels.  At panel cb the
// rows that take part are the panel's 16 diagonal rows, the block's rows below
// them and Z's rows up to the panel: always 16 + 64.  Per panel:
//   1. wavefront w updates rows 16 w.. of the panel (block rows when w >= cb,
//      Z rows when w < cb) by all earlier panels, on the matrix cores
//      (left-looking: one 16 x 16 tile per wavefront, inner dimension c0);
//   2. wavefronts 0 and 1 each hold the 16 diagonal rows (lanes 0..15, the
//      same in both) and half of the 64 other rows (lanes 16..47), one row
//      per lane and the 16 columns in registers, and run the 16 pivots without
//      touching LDS: the multipliers L[k][j] are read from lane k with
//      readlane, and the next pivot is formed before the other updates.
// Measured on N = 3 072 (48 dependent blocks): see potrf_batch_g.
template <class T>
__device__ __forceinline__ void diag_factor(DiagSmem &sm, int nb, T *__restrict__ A, int64_t lda, int64_t k0,
                                            T *__restrict__ Linv, T *__restrict__ LinvT, int32_t *flag,
                                            int64_t *aux) {
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  bool bad = false;
#pragma unroll 1
  for (int cb = 0; cb < 4; cb++) {
    const int c0 = 16 * cb;
    if (cb > 0) {
      if (wv < 4) {
        // tile rows R = 16 wv.., columns c0..: minus sum_k rows[R][k] L[c][k]
        const int l15 = lane & 15, kq = lane >> 4;
        const int R = 16 * wv + l15;
        f64x4 acc = f64x4{0.0, 0.0, 0.0, 0.0};
        // a Z row has columns from its own block on: that block holds L below
        // the diagonal, Z above it and Z's diagonal in dinv
        const double dR = sm.dinv[R];
        const bool zrow = wv < cb;
        for (int kb = zrow ? wv : 0; kb < cb; kb++) {
#pragma unroll
          for (int s4 = 0; s4 < 4; s4++) {
            const int k = 16 * kb + 4 * s4 + kq;
            double av = sm.L[R][k];
            const double bv = sm.L[c0 + l15][k];
            if (zrow && kb == wv) av = k > R ? av : (k == R ? dR : 0.0);
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, acc, 0, 0, 0);
          }
        }
        // (a diagonal row's entries above the diagonal are never used)
#pragma unroll
        for (int i = 0; i < 4; i++) sm.L[16 * wv + 4 * i + kq][c0 + l15] -= acc[i];
      }
      __syncthreads();
    }
    double v[16];
    // row of this lane: lanes 0..15 the diagonal rows, lanes 16..47 rows
    // 32 wv.. of the 64 others (a Z row of the diagonal block starts as a row
    // of the identity); lanes 48..63 repeat lanes 32..47
    const int R = lane < 16 ? c0 + lane : 32 * (wv & 1) + (lane < 48 ? lane - 16 : lane - 32);
    const int d = R - c0;
    const bool unit = lane >= 16 && (unsigned)d < 16u;
    if (wv < 2) {
#pragma unroll
      for (int k = 0; k < 16; k++) {
        const double a = sm.L[R][c0 + k];
        v[k] = unit ? (k == d ? 1.0 : 0.0) : a;
      }
    }
    __syncthreads();
    if (wv < 2) {
      double piv = read_lane(v[0], 0);
#pragma unroll
      for (int j = 0; j < 16; j++) {
        if (!(piv > 0.0)) {
          bad = true;
          piv = 1.0;
        }
        const double rs = rsqrt(piv);
        v[j] *= rs;  // L[r][j]; at the pivot sqrt(piv); Z[r][j] on the identity's rows
        if (j + 1 < 16) piv = read_lane(fma(-v[j], v[j], v[j + 1]), j + 1);
#pragma unroll
        for (int k = j + 1; k < 16; k++) v[k] = fma(-v[j], read_lane(v[j], k), v[k]);
      }
      if (lane < 48) {
        double dg = 0.0;
#pragma unroll
        for (int k = 0; k < 16; k++) {
          // block rows below the panel and Z rows above it: every column;
          // diagonal rows: L up to the diagonal (wavefront 0); Z rows of the
          // diagonal block: above it, the diagonal to dinv
          const bool put = lane < 16 ? (wv == 0 && k <= d) : (!unit || k > d);
          if (put) sm.L[R][c0 + k] = v[k];
          dg = k == d ? v[k] : dg;
        }
        if (unit) sm.dinv[R] = dg;
      }
    }
    __syncthreads();
  }
  if (bad && lane == 0 && wv == 0) {
    set_flag(flag, FPDE_ENOTSPD);
    atomicCAS((unsigned long long *)aux, ~0ull, (unsigned long long)k0);
  }
  // L to A (lower part inside the matrix), X = inv(L) row-major to Linv, X^T to LinvT
  if (tid >= 256) return;
#pragma unroll 8
  for (int it = 0; it < 16; it++) {
    const int idx = tid + 256 * it, r = idx >> 6, m = idx & 63;
    const double lrm = sm.L[r][m], lmr = sm.L[m][r], dr = sm.dinv[r];
    if (r < nb && m < nb && m <= r) A[(k0 + r) * lda + k0 + m] = (T)lrm;
    Linv[idx] = (T)((m < r) ? lmr : ((m == r) ? dr : 0.0));   // X[r][m]
    LinvT[idx] = (T)((r < m) ? lrm : ((m == r) ? dr : 0.0));  // X[m][r]
  }
}

}  // namespace fpde
