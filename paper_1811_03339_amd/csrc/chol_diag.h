// Factorization of one 64 x 64 diagonal block of the blocked Cholesky in
// LDS (256 threads), shared by the first-panel kernel and the trailing
// updates whose tile (0, 0) factors the next diagonal block.
#pragma once

#include "dense.h"

namespace fpde {

// LDS used by one diagonal-block factorization: the block on entry (lower
// part, zeros above; identity past the matrix end); L replaces it in the
// lower triangle, and Z = inv(L)^T fills the 16 x 16 tiles above the diagonal
// ones.  Z's diagonal tile of panel p is in Zd[p & 1] until panel p + 2.
struct DiagSmem {
  double L[NB][NB + 1];
  double Zd[2][16][17];
  double none[64 + 16];  // where lanes without a row of their own write
};

// 1 / sqrt(x) from the hardware's estimate and one third-order step of the
// series of (1 - t)^(-1/2), t = 1 - x y^2; NaN for x < 0, 0 for infinite x
__device__ __forceinline__ double rsqrt_step(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double t = fma(-((x < INFINITY ? x : 0.0) * y), y, 1.0);
  return fma(y * t, fma(t, 0.375, 0.5), y);
}

// rows 16 w.., columns 16 J.. of the block (and of Z) -= panel p's part, for
// one wavefront: rows of the block (w > p) or of Z (w <= p).  Entries above
// the diagonal of the block's diagonal tiles come out meaningless and unused.
__device__ __forceinline__ void diag_tile_update(DiagSmem &sm, int w, int J, int p) {
  const int lane = threadIdx.x & 63, l15 = lane & 15, kq = lane >> 4;
  const double *a = w == p ? &sm.Zd[p & 1][l15][0] : &sm.L[16 * w + l15][16 * p];
  double av[4], bv[4], c[4];
#pragma unroll
  for (int q = 0; q < 4; q++) {
    av[q] = a[4 * q + kq];
    bv[q] = sm.L[16 * J + l15][16 * p + 4 * q + kq];
    c[q] = sm.L[16 * w + 4 * q + kq][16 * J + l15];
  }
  f64x4 acc = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int q = 0; q < 4; q++) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av[q], bv[q], acc, 0, 0, 0);
#pragma unroll
  for (int q = 0; q < 4; q++) sm.L[16 * w + 4 * q + kq][16 * J + l15] = c[q] - acc[q];
}

// panel p's columns of L to A's block at (k0, k0) and of inv(L) to Linv
// (rows) and LinvT, by wavefront w of nw (1, 2 or 4)
template <class T>
__device__ __forceinline__ void diag_store_panel(const DiagSmem &sm, int p, int w, int nw, int nb, T *__restrict__ A,
                                                 int64_t lda, int64_t k0, T *__restrict__ Linv,
                                                 T *__restrict__ LinvT) {
  const int lane = threadIdx.x & 63;
  const int c = lane & 15;
  // four rows of sixteen columns, and one column of 64 rows, a step; four
  // steps' reads of the block before their stores
#pragma unroll 1
  for (int i0 = w; i0 < 16; i0 += 4 * nw) {
    double v[4], z[4], vt[4], zt[4];
#pragma unroll
    for (int q = 0; q < 4; q++) {
      const int i = i0 + q * nw;
      const int r = 4 * i + (lane >> 4);
      v[q] = sm.L[r][16 * p + c];
      z[q] = sm.Zd[p & 1][r & 15][c];
      vt[q] = sm.L[lane][16 * p + i];
      zt[q] = sm.Zd[p & 1][lane & 15][i];
    }
#pragma unroll
    for (int q = 0; q < 4; q++) {
      const int i = i0 + q * nw;
      const int r = 4 * i + (lane >> 4), rel = (r >> 4) - p, relt = (lane >> 4) - p;
      LinvT[r * NB + 16 * p + c] = (T)(rel < 0 ? v[q] : (rel == 0 ? z[q] : 0.0));
      Linv[(16 * p + i) * NB + lane] = (T)(relt < 0 ? vt[q] : (relt == 0 ? zt[q] : 0.0));
      if (r < nb && 16 * p + c <= r) A[(k0 + r) * lda + k0 + 16 * p + c] = (T)v[q];
    }
  }
}

// Factor the 64 x 64 diagonal block held in sm.L (rows/columns >= nb are
// identity), write L over A's block at (k0, k0), inv(L) to Linv and
// inv(L)^T to LinvT.  The first 256 threads of the workgroup work; further
// threads only take part in its barriers.
//
// What bounds it is the dependent chain of 64 pivots, so everything else is
// kept off that chain.  The column operations that turn the block into L turn
// the identity below it into Z = inv(L)^T, so the two are factored together as
// one tall matrix in 16-column panels.  At panel cb the rows that take part
// are the panel's 16 diagonal rows, the block's rows below them and Z's rows
// up to the panel: always 16 + 64.  Per panel:
//   1. wavefront w updates rows 16 w.. of the panel by panel cb - 1 (one
//      16 x 16 tile on the matrix cores; earlier panels are applied already);
//   2. wavefronts 0 and 1 each hold the 16 diagonal rows (lanes 0..15, the
//      same in both) and half of the 64 other rows (lanes 16..47), one row
//      per lane and the 16 columns in registers, and run the pivots two at a
//      time without touching LDS: the multipliers L[k][j] are read from lane k
//      with readlane, and the second pivot c - (b / sqrt(a))^2 of a pivot block
//      [a b; b c] is formed beside the first one's column, from the same rounded
//      numbers that the column holds (from a c - b^2, which does not wait for the
//      first root, the error of L L^T grew with the pair's condition);
//   3. beside them wavefronts 2 and 3 apply panel cb - 1 to the columns right
//      of the panel and write its outputs.
// One wavefront factoring a 16-column block at a time through LDS and four
// barriers per block took 30 us a block; the chain in registers 21 us, with the
// pivots in pairs and the rest beside them 12 us (kernel k_potrf_diag, 64 rows).
template <class T>
__device__ __forceinline__ void diag_factor(DiagSmem &sm, int nb, T *__restrict__ A, int64_t lda, int64_t k0,
                                            T *__restrict__ Linv, T *__restrict__ LinvT, int32_t *flag,
                                            int64_t *aux) {
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  bool good = true;
#pragma unroll 1
  for (int cb = 0; cb < 4; cb++) {
    const int c0 = 16 * cb;
    if (cb > 0) {
      if (wv < 4) diag_tile_update(sm, wv, cb, cb - 1);
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
      for (int k = 0; k < 16; k++) v[k] = sm.L[R][c0 + k];
#pragma unroll
      for (int k = 0; k < 16; k++) v[k] = unit ? (k == d ? 1.0 : 0.0) : v[k];
    }
    __syncthreads();  // both wavefronts hold the diagonal rows
    if (wv < 2) {
      double a = read_lane(v[0], 0), b = read_lane(v[0], 1), c = read_lane(v[1], 1);
#pragma unroll
      for (int j = 0; j < 16; j += 2) {
        const double ra = rsqrt_step(a), l21 = b * ra, a2 = fma(-l21, l21, c);
        good = good && a > 0.0 && a2 > 0.0;
        const double rd = rsqrt_step(a2);  // 1 / L[j+1][j+1]
        v[j] *= ra;
        v[j + 1] = fma(-v[j], l21, v[j + 1]) * rd;
#pragma unroll
        for (int k = j + 2; k < 16; k++) {
          v[k] = fma(-v[j + 1], read_lane(v[j + 1], k), fma(-v[j], read_lane(v[j], k), v[k]));
          if (k == j + 3) {  // the next pivot block, as soon as it is there
            a = read_lane(v[j + 2], j + 2);
            b = read_lane(v[j + 2], j + 3);
            c = read_lane(v[j + 3], j + 3);
          }
        }
      }
      double *to = lane >= 48 || (lane < 16 && wv == 1) ? &sm.none[lane]
                                                        : (unit ? &sm.Zd[cb & 1][d][0] : &sm.L[R][c0]);
#pragma unroll
      for (int k = 0; k < 16; k++) to[k] = v[k];
    } else if (wv < 4 && cb > 0) {
      // tiles (row block w, column block J > cb) that panel cb - 1 reaches:
      // Z rows w < cb and block rows w >= J
#pragma unroll 1
      for (int J = cb + 1; J < 4; J++)
        for (int w = 0; w < 4; w++)
          if ((w < cb || w >= J) && ((w ^ J ^ wv) & 1) == 0) diag_tile_update(sm, w, J, cb - 1);
      diag_store_panel(sm, cb - 1, wv - 2, 2, nb, A, lda, k0, Linv, LinvT);
    }
    __syncthreads();
  }
  if (!good && lane == 0 && wv == 0) {
    set_flag(flag, FPDE_ENOTSPD);
    atomicCAS((unsigned long long *)aux, ~0ull, (unsigned long long)k0);
  }
  if (wv < 4) diag_store_panel(sm, 3, wv, 4, nb, A, lda, k0, Linv, LinvT);
}

}  // namespace fpde
