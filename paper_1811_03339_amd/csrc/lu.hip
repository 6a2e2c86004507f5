// Dense LU factorization without pivoting, A = L U (L unit lower, U upper,
// both kept in A), and the solve A u = b, for the non-symmetric matrix of
// the divergence-form two-sided problem (Sec. 3).  Its bilinear form is
// coercive (the symmetric part of -A is positive definite), so every leading
// block is nonsingular and no row exchange is needed; a zero or non-finite
// pivot is reported, not worked around.
//
// Blocked right-looking, panel width NB = 64, panels in groups of kLuGroup:
//   diag   : one workgroup factors A_kk = L_kk U_kk and forms inv(L_kk) and
//            inv(U_kk); for every panel after the first this runs inside the
//            preceding update (its tile (0, 0));
//   panels : L_ik = A_ik inv(U_kk) for every 64-row strip below and
//            U_kj = inv(L_kk) A_kj for every 64-column strip to the right,
//            each a 64 x 64 x 64 tile product (no sequential dependency);
//   update : inside a group, C_ij -= L_ik U_kj over the group's later block
//            columns and block rows (64 x 64 tiles); after its last panel, the
//            trailing square once by the whole group (128 x 128 tiles).
// The solve runs the block-row triangular solves of dense.h forward with L
// (inv(L_bb) per block) and backward with U (inv(U_bb)).
#include <cmath>

#include "dense.h"

namespace fpde {

namespace {

struct LuInvSmem {
  double row[2][2][NB];  // [buffer][factor | inverse][column]: the pivot row
  double col[2][NB];     // [buffer][row]: the pivot column
};

// inv(L) and inv(U) of an existing factor's 64 x 64 diagonal block.  Thread t
// owns row r = t >> 2 of the block and 16 of its columns (the four threads of a
// row are neighbouring lanes of one wavefront): a holds L (strict lower, unit
// diagonal) + U (upper); on exit y = inv(L) and z = inv(U) in the same layout.
// Rows/columns past nb are identity.
//
// One pass over the columns j = 0..63, one barrier each: row j and column j
// are published to LDS (two alternating buffers, so the next step's writes
// cannot overtake this step's reads), then
//   rows r > j:  Y_rc -= L_rj Y_jc (Y = I at the start, inv(L) at the end);
//   rows r <= j: column j of W = inv(U) from W U = I,
//                W_rj = (delta_rj - sum_{k<j} W_rk U_kj) / U_jj, whose
//                column of U is the published column j and whose W_rk were
//                formed at the earlier steps (a 4-lane sum over the row's
//                threads).
// The columns run in 16 blocks of 4 (a runtime loop over the blocks, the 4
// steps of a block unrolled), so the code stays small.  To keep register
// indices static, the three arrays rotate by one slot after each block: in
// block kb, slot s of a thread with t & 3 = cl holds column
// cl + 4 ((s + kb) mod 16), so the block's own columns are in slot 0.  The
// LDS row buffer is kept in slot order; the column buffer (indexed by row)
// in the same rotated order, row r at (r & 3) + 4 ((r / 4 - kb) mod 16).
__device__ __forceinline__ void lu_block_inverses(LuInvSmem &sm, double (&a)[16], double (&y)[16], double (&z)[16]) {
  const int tid = threadIdx.x, r = tid >> 2, cls = tid & 3;
#pragma unroll
  for (int k = 0; k < 16; k++) {
    y[k] = (cls + 4 * k == r) ? 1.0 : 0.0;
    z[k] = 0.0;
  }
#pragma unroll 1
  for (int kb = 0; kb < 16; kb++) {
    const int own = (r & 3) + 4 * (((r >> 2) - kb) & 15);  // this row's slot in the column buffer
    const int live = 15 - kb;  // slots 1..live hold columns right of the block
#pragma unroll
    for (int c = 0; c < 4; c++) {
      const int j = 4 * kb + c, buf = c & 1;
      if (r == j) {
#pragma unroll
        for (int s = 0; s < 16; s++) {
          sm.row[buf][0][cls + 4 * s] = a[s];
          sm.row[buf][1][cls + 4 * s] = y[s];
        }
      }
      if (cls == c) sm.col[buf][own] = a[0];
      __syncthreads();
      // everything this step reads from LDS, loaded before any use
      double ry[16], rc[16];
#pragma unroll
      for (int s = 0; s < 16; s++) {
        ry[s] = sm.row[buf][1][cls + 4 * s];
        rc[s] = sm.col[buf][cls + 4 * s];
      }
      const double piv = sm.row[buf][0][c];  // U_jj: column j is slot 0 of lane class c
      const double cown = sm.col[buf][own];
      const double rp = 1.0 / piv;
      // column j of inv(U): sum over the columns left of j (inactive slots
      // contribute an exact zero)
      double part = 0.0;
#pragma unroll
      for (int s = 0; s < 16; s++) {
        const bool left = s == 0 ? cls < c : s > live;
        part = fma(left ? z[s] : 0.0, rc[s], part);
      }
      part += __shfl_xor(part, 1, 64);
      part += __shfl_xor(part, 2, 64);
      if (cls == c && r <= j) z[0] = ((r == j ? 1.0 : 0.0) - part) * rp;
      // elimination below the diagonal: multipliers are zero where a slot does
      // not take part, which leaves it unchanged
      const double l = r > j ? cown : 0.0;
#pragma unroll
      for (int s = 0; s < 16; s++) {
        const bool right = s == 0 ? cls > c : s <= live;
        y[s] = fma(right ? 0.0 : -l, ry[s], y[s]);
      }
    }
    // rotate: slot s takes slot s + 1, slot 15 takes slot 0
    const double a0 = a[0], y0 = y[0], z0 = z[0];
#pragma unroll
    for (int s = 0; s < 15; s++) {
      a[s] = a[s + 1];
      y[s] = y[s + 1];
      z[s] = z[s + 1];
    }
    a[15] = a0;
    y[15] = y0;
    z[15] = z0;
  }
}

// One workgroup per diagonal block b of an existing factor: inv(L_bb)^T and
// inv(U_bb)^T for the triangular solves.
__global__ void __launch_bounds__(256) k_lu_inverses(const double *__restrict__ A, int64_t lda, int64_t n,
                                                     double *__restrict__ LinvT, double *__restrict__ UinvT) {
  __shared__ LuInvSmem sm;
  const int64_t b = blockIdx.x;
  const int64_t k0 = b * NB;
  const int nb = (int)((n - k0) < NB ? (n - k0) : NB);
  const int tid = threadIdx.x, r = tid >> 2, cls = tid & 3;
  double a[16], y[16], z[16];
  const int rr = r < nb ? r : nb - 1;
#pragma unroll
  for (int k = 0; k < 16; k++) {
    const int c = cls + 4 * k;
    a[k] = A[(k0 + rr) * lda + k0 + (c < nb ? c : nb - 1)];
  }
#pragma unroll
  for (int k = 0; k < 16; k++) {
    const int c = cls + 4 * k;
    if (r >= nb || c >= nb) a[k] = (r == c) ? 1.0 : 0.0;
  }
  lu_block_inverses(sm, a, y, z);
  const int64_t o = b * NB * NB;
#pragma unroll
  for (int k = 0; k < 16; k++) {
    const int c = cls + 4 * k;
    LinvT[o + c * NB + r] = y[k];
    UinvT[o + c * NB + r] = z[k];
  }
}

// ---- Factorization of one 64 x 64 diagonal block, 512 threads ----
//
// The column operations that turn the block A into L turn the identity below
// it into inv(U), and those that turn A^T into U^T turn the identity into
// inv(L)^T.  The two tall matrices are factored side by side in 16-column
// panels (problem 0: A, problem 1: A^T), each by two wavefronts that hold one
// row per lane: the panel's 16 diagonal rows (lanes 0..15, the same in both)
// and half of the 64 other rows (lanes 16..47: the rows below the panel and
// the inverse's rows up to it).  The 16 pivots of a panel then run in
// registers, the pivot row's entries read with readlane; the four other
// wavefronts apply the previous panel to the columns right of the current one
// (16 x 16 tiles on the matrix cores) and write its outputs.  The chain of 64
// dependent reciprocals is what bounds it: 20 us a first block.  One pass over
// the pivots with one row in four threads and a barrier per pivot took 72 us.
struct LuSmem {
  double M[NB][NB + 1];      // the block; L and U replace it outside the diagonal tiles
  double Zt[12][16][17];     // off-diagonal tiles: inv(U) above the diagonal, inv(L) below
  double Zd[2][2][16][17];   // [problem][panel & 1]: diagonal tiles of inv(U), inv(L)^T
  double D[2][2][16][17];    // [problem][panel & 1]: diagonal rows of L, U^T
  double none[64 + 16];      // where lanes without a row of their own write
};

__device__ __forceinline__ int lu_tile(int w, int J) { return 3 * w + (J > w ? J - 1 : J); }

// problem s, row block w, column block J: minus panel p's part
__device__ __forceinline__ void lu_tile_update(LuSmem &sm, int s, int w, int J, int p) {
  const int lane = threadIdx.x & 63, l15 = lane & 15, kq = lane >> 4;
  // operand rows 16 w + l15 over the panel's columns, and the result's place,
  // as (base, stride) of the problem's own orientation
  const double *a;
  int as;
  if (w == p) {
    a = &sm.Zd[s][p & 1][l15][kq];
    as = 1;
  } else if (w > p) {
    a = s ? &sm.M[16 * p + kq][16 * w + l15] : &sm.M[16 * w + l15][16 * p + kq];
    as = s ? NB + 1 : 1;
  } else {
    a = s ? &sm.Zt[lu_tile(p, w)][kq][l15] : &sm.Zt[lu_tile(w, p)][l15][kq];
    as = s ? 17 : 1;
  }
  const double *b = s ? &sm.M[16 * J + l15][16 * p + kq] : &sm.M[16 * p + kq][16 * J + l15];
  const int bs = s ? 1 : NB + 1;
  double *c;
  int cs;
  if (w >= J) {
    c = s ? &sm.M[16 * J + l15][16 * w + kq] : &sm.M[16 * w + kq][16 * J + l15];
    cs = s ? 1 : NB + 1;
  } else {
    c = s ? &sm.Zt[lu_tile(J, w)][l15][kq] : &sm.Zt[lu_tile(w, J)][kq][l15];
    cs = s ? 1 : 17;
  }
  double av[4], bv[4], cv[4];
#pragma unroll
  for (int q = 0; q < 4; q++) {
    av[q] = a[4 * q * as];
    bv[q] = b[4 * q * bs];
    cv[q] = c[4 * q * cs];
  }
  f64x4 acc = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int q = 0; q < 4; q++) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av[q], bv[q], acc, 0, 0, 0);
  // the first panel that reaches a tile of the inverses finds no value there
#pragma unroll
  for (int q = 0; q < 4; q++) c[4 * q * cs] = (w == p ? 0.0 : cv[q]) - acc[q];
}

// panel p's rows of U and columns of L to A's block at (k0, k0), its rows of
// inv(L) to Linv and LinvT and its columns of inv(U) to UinvT, by wavefront w
// of nw (a power of two)
__device__ __forceinline__ void lu_store_panel(const LuSmem &sm, int p, int w, int nw, int nb, double *__restrict__ A,
                                               int64_t lda, int64_t k0, double *__restrict__ Linv,
                                               double *__restrict__ LinvT, double *__restrict__ UinvT) {
  const int lane = threadIdx.x & 63, l15 = lane & 15, q = p & 1;
#pragma unroll 2
  for (int i = w; i < 16; i += nw) {
    {  // rows r (four of them), panel column l15
      const int r = 4 * i + (lane >> 4), br = r >> 4, c = 16 * p + l15;
      const double d = l15 < (r & 15) ? sm.D[0][q][r & 15][l15] : sm.D[1][q][l15][r & 15];
      const double v = br == p ? d : sm.M[r][c];
      if (br >= p && r < nb && c < nb) A[(k0 + r) * lda + k0 + c] = v;
      // inv(L)[16 p + l15][r]
      const double z = br < p ? sm.Zt[lu_tile(p, br < p ? br : 0)][l15][r & 15] : sm.Zd[1][q][r & 15][l15];
      LinvT[r * NB + c] = br <= p ? z : 0.0;
    }
    {  // panel row i, every column (lane)
      const int bc = lane >> 4, r = 16 * p + i, ct = bc < p ? bc : 0;
      if (bc > p && r < nb && lane < nb) A[(k0 + r) * lda + k0 + lane] = sm.M[r][lane];
      const double zl = bc < p ? sm.Zt[lu_tile(p, ct)][i][l15] : sm.Zd[1][q][l15][i];
      Linv[r * NB + lane] = bc <= p ? zl : 0.0;
      // inv(U)[lane][16 p + i]
      const double zu = bc < p ? sm.Zt[lu_tile(ct, p)][l15][i] : sm.Zd[0][q][l15][i];
      UinvT[r * NB + lane] = bc <= p ? zu : 0.0;
    }
  }
}

// 1 / x from the hardware's estimate and two Newton steps
__device__ __forceinline__ double rcp_step(double x) {
  double y = __builtin_amdgcn_rcp(x);
  y = fma(fma(-x, y, 1.0), y, y);
  return fma(fma(-x, y, 1.0), y, y);
}

// Factor the block held in sm.M (rows/columns >= nb are identity) and write
// its outputs (the four sets of block k0 / 64, the inverse sets given at that
// block).  All 512 threads.
__device__ __forceinline__ void lu_diag_factor(LuSmem &sm, int nb, double *__restrict__ A, int64_t lda, int64_t k0,
                                               double *__restrict__ Linv, double *__restrict__ LinvT,
                                               double *__restrict__ UinvT, int32_t *flag, int64_t *aux) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  bool good = true;
#pragma unroll 1
  for (int cb = 0; cb < 4; cb++) {
    const int c0 = 16 * cb;
    if (cb > 0) {
      // the seven tiles of this panel's columns (the diagonal tile is shared)
      if (wv < 4) lu_tile_update(sm, 0, wv, cb, cb - 1);
      else if (wv - 4 != cb) lu_tile_update(sm, 1, wv - 4, cb, cb - 1);
      __syncthreads();
    }
    const int s = (wv >> 1) & 1, half = wv & 1;
    const int R = lane < 16 ? c0 + lane : 32 * half + (lane < 48 ? lane - 16 : lane - 32);
    const int d = R - c0, wr = R >> 4, wz = wr < cb ? wr : (cb ? 0 : 1);
    const bool unit = lane >= 16 && (unsigned)d < 16u;
    // this lane's row of the panel: where it is read and, after the pivots, written
    double *row;
    int rs;
    if (R < c0) {
      row = s ? &sm.Zt[lu_tile(cb, wz)][0][R & 15] : &sm.Zt[lu_tile(wz, cb)][R & 15][0];
      rs = s ? 17 : 1;
    } else {
      row = s ? &sm.M[c0][R] : &sm.M[R][c0];
      rs = s ? NB + 1 : 1;
    }
    double v[16];
    if (wv < 4) {
#pragma unroll
      for (int k = 0; k < 16; k++) v[k] = row[k * rs];
#pragma unroll
      for (int k = 0; k < 16; k++) v[k] = unit ? (k == d ? 1.0 : 0.0) : v[k];
    }
    __syncthreads();
    if (wv < 4) {
      // L = v[j] / pivot in A, row j's entries / pivot in its transpose: from an
      // entry of the block both problems take the product of the same two
      // numbers, so that they agree in every bit.  (With v[j] / pivot in both,
      // the pivots, and so L U, were off by the rounding times the condition of
      // the unknowns before them.)  A loop for each: 1728 unknowns 1002 us; with
      // a branch per pivot, across which nothing is scheduled, 1027.
      double piv = read_lane(v[0], 0);
      if (s == 0) {
#pragma unroll
        for (int j = 0; j < 16; j++) {
          good = good && fabs(piv) > 0.0 && fabs(piv) < INFINITY;
          v[j] *= rcp_step(piv);
#pragma unroll
          for (int k = j + 1; k < 16; k++) v[k] = fma(-v[j], read_lane(v[k], j), v[k]);
          if (j < 15) piv = read_lane(v[j + 1], j + 1);
        }
      } else {
#pragma unroll
        for (int j = 0; j < 16; j++) {
          const double r = rcp_step(piv);
#pragma unroll
          for (int k = j + 1; k < 16; k++) v[k] = fma(-v[j], read_lane(v[k], j) * r, v[k]);
          if (j < 15) piv = read_lane(v[j + 1], j + 1);
        }
      }
      if (lane >= 48 || (lane < 16 && half)) {
        row = &sm.none[lane];
        rs = 1;
      } else if (lane < 16) {
        row = &sm.D[s][cb & 1][lane][0];
        rs = 1;
      } else if (unit) {
        row = &sm.Zd[s][cb & 1][d][0];
        rs = 1;
      }
#pragma unroll
      for (int k = 0; k < 16; k++) row[k * rs] = v[k];
    } else if (cb > 0) {
      const int p = cb - 1;
      int i = 0;
#pragma unroll 1
      for (int J = cb + 1; J < 4; J++)
#pragma unroll 1
        for (int x = 0; x < 8; x++) {
          const int ps = x >> 2, w = x & 3;
          if ((w <= p || w >= J) && !(ps == 1 && w == J) && (i++ & 3) == wv - 4) lu_tile_update(sm, ps, w, J, p);
        }
      lu_store_panel(sm, p, wv - 4, 4, nb, A, lda, k0, Linv, LinvT, UinvT);
    }
    __syncthreads();
  }
  if (!good && lane == 0 && wv == 0) {
    set_flag(flag, FPDE_ESINGULAR);
    atomicCAS((unsigned long long *)aux, ~0ull, (unsigned long long)k0);
  }
  lu_store_panel(sm, 3, wv, 8, nb, A, lda, k0, Linv, LinvT, UinvT);
}

// the first diagonal block on its own (block 0 of the inverse sets)
__global__ void __launch_bounds__(512) k_lu_diag(double *__restrict__ A, int64_t lda, int64_t n,
                                                 double *__restrict__ Linv, double *__restrict__ LinvT,
                                                 double *__restrict__ UinvT, int32_t *flag, int64_t *aux) {
  extern __shared__ char lu_lds[];
  LuSmem &sm = *(LuSmem *)lu_lds;
  const int nb = (int)(n < NB ? n : NB);
  double av[8];
#pragma unroll
  for (int it = 0; it < 8; it++) {
    const int idx = threadIdx.x + 512 * it, r = idx >> 6, c = idx & 63;
    av[it] = A[(r < nb ? r : nb - 1) * lda + (c < nb ? c : nb - 1)];
  }
#pragma unroll
  for (int it = 0; it < 8; it++) {
    const int idx = threadIdx.x + 512 * it, r = idx >> 6, c = idx & 63;
    sm.M[r][c] = r < nb && c < nb ? av[it] : (r == c ? 1.0 : 0.0);
  }
  __syncthreads();
  lu_diag_factor(sm, nb, A, lda, 0, Linv, LinvT, UinvT, flag, aux);
}

// out = P Q over a 64-deep inner dimension: P is 64 x 64 (rows past `prow`
// read as zero), Q is 64 x 64 row-major by inner index (columns past `qcol`
// read as zero).  Two 32-deep chunks staged through LDS as in tile_product (Q
// transposed on the way in, every load at a valid address), multiplied on
// the matrix cores; value q of a thread's 16 sits at (frag_row<double>(q),
// frag_col<double>(q)).
template <int KD = NB>
__device__ __forceinline__ void tile_nn(const double *__restrict__ P, int64_t ldp, int prow,
                                        const double *__restrict__ Q, int64_t ldq, int qcol, double (*sP)[33],
                                        double (*sQ)[33], double out[16]) {
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int lc = tid & 31, lr = tid >> 5;  // P: rows lr + 8 it, column lc of a chunk
  const int qc = tid & 63, qr = tid >> 6;  // Q: column qc, inner rows qr + 4 it of a chunk
  const int qcc = qc < qcol ? qc : qcol - 1;
  const int rm = 32 * (w >> 1) + (lane & 15), cm = 32 * (w & 1) + (lane & 15), kq = lane >> 4;
  f64x4 acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; a++)
#pragma unroll
    for (int b = 0; b < 2; b++) acc[a][b] = f64x4{0.0, 0.0, 0.0, 0.0};
  double pr[8], qv[8];
  auto load = [&](int kk) {
#pragma unroll
    for (int it = 0; it < 8; it++) {
      const int rr = lr + 8 * it;
      pr[it] = P[(int64_t)(rr < prow ? rr : prow - 1) * ldp + kk + lc];
      qv[it] = Q[(int64_t)(kk + qr + 4 * it) * ldq + qcc];
    }
  };
  load(0);
#pragma unroll
  for (int kk = 0; kk < KD; kk += 32) {
#pragma unroll
    for (int it = 0; it < 8; it++) {
      const int rr = lr + 8 * it;
      sP[rr][lc] = rr < prow ? pr[it] : 0.0;
      sQ[qc][qr + 4 * it] = qc < qcol ? qv[it] : 0.0;
    }
    __syncthreads();
    if (kk + 32 < KD) load(kk + 32);
    mfma_chunk(sP, sQ, rm, cm, kq, acc);
    __syncthreads();
  }
  mfma_out(acc, out);
}

// Workgroups [0, ns): L strips (rows k1 + 64 x, columns of panel k);
// [ns, 2 ns): U strips (rows of panel k, columns k1 + 64 (x - ns)).
__global__ void __launch_bounds__(256) k_lu_panels(double *__restrict__ A, int64_t lda, int64_t n, int64_t k0,
                                                   int ns, const double *__restrict__ Linv_k,
                                                   const double *__restrict__ UinvT_k) {
  __shared__ double sP[64][33], sQ[64][33];
  const int64_t k1 = k0 + NB;
  const int x = blockIdx.x;
  double out[16];
  if (x < ns) {
    const int64_t r0 = k1 + 64 * (int64_t)x;
    const int rows = (int)((n - r0) < 64 ? (n - r0) : 64);
    tile_product(A + r0 * lda + k0, lda, rows, UinvT_k, NB, NB, sP, sQ, out);
#pragma unroll
    for (int q = 0; q < 16; q++) {
      const int rr = frag_row<double>(q);
      if (rr < rows) A[(r0 + rr) * lda + k0 + frag_col<double>(q)] = out[q];
    }
  } else {
    const int64_t c0 = k1 + 64 * (int64_t)(x - ns);
    const int cols = (int)((n - c0) < 64 ? (n - c0) : 64);
    tile_nn(Linv_k, NB, NB, A + k0 * lda + c0, lda, cols, sP, sQ, out);
#pragma unroll
    for (int q = 0; q < 16; q++) {
      const int cc = frag_col<double>(q);
      if (cc < cols) A[(k0 + frag_row<double>(q)) * lda + c0 + cc] = out[q];
    }
  }
}

// ---- Updates C -= L U, eight wavefronts per tile ----
//
// Tiles of TM x TM (64 inside a group, 128 for the trailing square) over an
// inner dimension KD in 16-deep chunks, double-buffered in LDS: rows of L
// padded to 17, rows of U (16 of them, TM wide) padded by 16 so that the two
// rows a half wavefront reads fall in different halves of the banks.
// Wavefront w of eight holds rows (TM / 2) (w >> 2).., columns (TM / 4) (w & 3)..
// of the tile: 128-wide tiles 64 x 32 each (64 accumulator registers, two
// workgroups per CU and four wavefronts per SIMD as in the FP64 Cholesky).
template <int TM>
struct LuGemmSmem {
  double a[2][TM][17];
  double b[2][16][TM + 16];
};

template <int TM, int KD>
__device__ __forceinline__ void lu_product(const double *__restrict__ P, const double *__restrict__ Q, int64_t lda,
                                           int prow, int qcol, LuGemmSmem<TM> &sm, f64x4 (&acc)[TM / 32][TM / 64]) {
  constexpr int AM = TM / 32, BN = TM / 64, NA = TM / 32, NBQ = TM / 32;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6, wr = w >> 2, wc = w & 3, l15 = lane & 15, kq = lane >> 4;
  const int pc = t & 15, pr = t >> 4;            // L: column pc, rows pr + 32 it
  constexpr int RQ = 512 / TM;                   // U: column qc, rows qr + RQ it
  const int qc = t & (TM - 1), qr = t / TM;
  int64_t po[NA];
#pragma unroll
  for (int it = 0; it < NA; it++) {
    const int r = pr + 32 * it;
    po[it] = (int64_t)(r < prow ? r : prow - 1) * lda + pc;
  }
  const int64_t qo = (int64_t)qr * lda + (qc < qcol ? qc : qcol - 1);
#pragma unroll
  for (int x = 0; x < AM; x++)
#pragma unroll
    for (int y = 0; y < BN; y++) acc[x][y] = f64x4{0.0, 0.0, 0.0, 0.0};
  double pv[NA], qv[NBQ];
  auto load = [&](int kk) {
#pragma unroll
    for (int it = 0; it < NA; it++) pv[it] = (P + kk)[po[it]];
#pragma unroll
    for (int it = 0; it < NBQ; it++) qv[it] = (Q + (int64_t)(kk + RQ * it) * lda)[qo];
  };
  auto put = [&](int buf) {
#pragma unroll
    for (int it = 0; it < NA; it++) sm.a[buf][pr + 32 * it][pc] = pr + 32 * it < prow ? pv[it] : 0.0;
#pragma unroll
    for (int it = 0; it < NBQ; it++) sm.b[buf][qr + RQ * it][qc] = qc < qcol ? qv[it] : 0.0;
  };
  load(0);
  put(0);
  __syncthreads();
#pragma unroll 1
  for (int kk = 0; kk < KD; kk += 16) {
    const int buf = (kk >> 4) & 1;
    const bool more = kk + 16 < KD;
    if (more) load(kk + 16);
#pragma unroll
    for (int k4 = 0; k4 < 16; k4 += 4) {
      double av[AM], bv[BN];
#pragma unroll
      for (int x = 0; x < AM; x++) av[x] = sm.a[buf][(TM / 2) * wr + 16 * x + l15][k4 + kq];
#pragma unroll
      for (int y = 0; y < BN; y++) bv[y] = sm.b[buf][k4 + kq][(TM / 4) * wc + 16 * y + l15];
#pragma unroll
      for (int x = 0; x < AM; x++)
#pragma unroll
        for (int y = 0; y < BN; y++) acc[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[x], bv[y], acc[x][y], 0, 0, 0);
    }
    if (more) put(buf ^ 1);
    __syncthreads();
  }
}

// C -= L U for tiles of the square from `base`, with L = columns and U = rows
// [k0, k0 + KD).  edge = 0: the whole square, T x T tiles taken in 8 x 8
// super-blocks dealt to the XCDs in contiguous ranges (an XCD's tiles share
// block rows of L and block columns of U in its L2).  edge > 0: the first
// `edge` tile columns (every row) and the first `edge` tile rows (the columns
// right of them): what the later panels of a group read.  The workgroup of tile
// (0, 0) keeps the next diagonal block, its top-left 64 x 64, and factors it at
// once, beside the rest of the update.
constexpr int kLuSuper = 8;
__host__ __device__ inline int64_t lu_items(int64_t T, int edge) {
  if (edge > 0) return edge >= T ? T * T : edge * T + edge * (T - edge);
  const int64_t S = (T + kLuSuper - 1) / kLuSuper;
  return S * S * kLuSuper * kLuSuper;
}

template <int TM, int KD>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4)))
k_lu_update(double *__restrict__ A, int64_t lda, int64_t n, int64_t k0, int64_t base, int64_t T, int edge,
            int64_t items, double *__restrict__ Linv, double *__restrict__ LinvT, double *__restrict__ UinvT,
            int32_t *flag, int64_t *aux) {
  extern __shared__ char lu_lds[];
  const int64_t per = gridDim.x / 8;  // the grid is a multiple of 8
  const int64_t x = (blockIdx.x % 8) * per + blockIdx.x / 8;
  if (x >= items) return;
  int64_t I, J;
  if (edge > 0) {
    if (edge >= T || x < edge * T) {
      I = x % T;
      J = x / T;
    } else {
      const int64_t y = x - edge * T;
      I = y % edge;
      J = edge + y / edge;
    }
  } else {
    const int64_t S = (T + kLuSuper - 1) / kLuSuper, sb = x / (kLuSuper * kLuSuper), si = x % (kLuSuper * kLuSuper);
    I = kLuSuper * (sb / S) + si / kLuSuper;
    J = kLuSuper * (sb % S) + si % kLuSuper;
    if (I >= T || J >= T) return;
  }
  const int64_t ri = base + TM * I, cj = base + TM * J;
  const int prow = (int)((n - ri) < TM ? (n - ri) : TM);
  const int qcol = (int)((n - cj) < TM ? (n - cj) : TM);
  constexpr int AM = TM / 32, BN = TM / 64;
  f64x4 acc[AM][BN];
  lu_product<TM, KD>(A + ri * lda + k0, A + k0 * lda + cj, lda, prow, qcol, *(LuGemmSmem<TM> *)lu_lds, acc);
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int fr = (TM / 2) * (w >> 2) + (lane >> 4), fc = (TM / 4) * (w & 3) + (lane & 15);
  LuSmem &dg = *(LuSmem *)lu_lds;
  // (0, 0): the wavefronts that hold the top-left 64 x 64
  const bool keep = x == 0 && (TM / 2) * (w >> 2) < NB && (TM / 4) * (w & 3) < NB;
  double *c0 = A + ri * lda + cj;
#pragma unroll
  for (int a = 0; a < AM; a++) {
    double cv[BN][4];
#pragma unroll
    for (int b = 0; b < BN; b++)
#pragma unroll
      for (int i = 0; i < 4; i++) {
        const int r = fr + 16 * a + 4 * i, c = fc + 16 * b;
        cv[b][i] = c0[(int64_t)(r < prow ? r : prow - 1) * lda + (c < qcol ? c : qcol - 1)];
      }
#pragma unroll
    for (int b = 0; b < BN; b++)
#pragma unroll
      for (int i = 0; i < 4; i++) {
        const int r = fr + 16 * a + 4 * i, c = fc + 16 * b;
        const double v = cv[b][i] - acc[a][b][i];
        if (keep) dg.M[r][c] = r < prow && c < qcol ? v : (r == c ? 1.0 : 0.0);
        else if (r < prow && c < qcol) c0[(int64_t)r * lda + c] = v;
      }
  }
  if (x != 0) return;
  __syncthreads();
  const int64_t o = base * NB;  // block base / 64 of each inverse set
  lu_diag_factor(dg, prow < NB ? prow : NB, A, lda, base, Linv + o, LinvT + o, UinvT + o, flag, aux);
}

inline unsigned blocks_of(int64_t n, int b = 256) { return (unsigned)((n + b - 1) / b); }

}  // namespace

// the three inverse sets of the LU blocks inside the mesh's buffer
static int lu_inverses(fpde_mesh *m, int64_t n, double **Linv, double **LinvT, double **UinvT) {
  void *lv = nullptr;
  FPDE_TRY(ensure_linv(m, n, sizeof(double), 3, &lv));
  const int64_t per = ((n + NB - 1) / NB) * NB * NB;
  *Linv = (double *)lv;
  *LinvT = *Linv + per;
  *UinvT = *LinvT + per;
  return FPDE_OK;
}

// Panels per group: the trailing square is read and written once per group.
// One factorization at N = 8 162: pairs of panels on 64-wide tiles with the
// diagonal blocks of 72 us 18.9 ms; groups of 4 on 128-wide tiles 12.0 ms, of 8
// 11.2 ms, now 10.9 (33 TFLOP/s; 128 steps of about 29 us are 3.7 ms of it).  Running the
// next group's panels beside the trailing update (its own stream) gained
// nothing: their tiles wait for the compute units that the update holds.
constexpr int kLuGroup = 8;

template <int TM, int KD>
static void launch_lu_update(double *A, int64_t lda, int64_t n, int64_t k0, int64_t base, int edge, double *Linv,
                             double *LinvT, double *UinvT, fpde_mesh *m, hipStream_t s) {
  const int64_t T = (n - base + TM - 1) / TM, items = lu_items(T, edge);
  constexpr size_t lds = sizeof(LuSmem) > sizeof(LuGemmSmem<TM>) ? sizeof(LuSmem) : sizeof(LuGemmSmem<TM>);
  k_lu_update<TM, KD><<<(unsigned)(8 * ((items + 7) / 8)), 512, lds, s>>>(A, lda, n, k0, base, T, edge, items, Linv,
                                                                         LinvT, UinvT, m->flag, m->flag_aux);
}

int lu_factor(fpde_mesh *m, double *A, int64_t lda, int64_t n, hipStream_t s) {
  double *Linv, *LinvT, *UinvT;
  FPDE_TRY(lu_inverses(m, n, &Linv, &LinvT, &UinvT));
  const long t = timer_begin(m, s, FPDE_STAGE_LU);
  k_lu_diag<<<1, 512, sizeof(LuSmem), s>>>(A, lda, n, Linv, LinvT, UinvT, m->flag, m->flag_aux);
  for (int64_t k0 = 0; k0 < n; k0 += kLuGroup * NB) {
    for (int sp = 0; sp < kLuGroup; sp++) {
      const int64_t ks = k0 + sp * NB, rest = n - ks - NB;
      if (rest <= 0) goto factored;  // the last diagonal block is factored
      const int64_t o = (ks / NB) * NB * NB;
      const int ns = (int)((rest + 63) / 64);
      k_lu_panels<<<2 * ns, 256, 0, s>>>(A, lda, n, ks, ns, Linv + o, UinvT + o);
      if (sp + 1 < kLuGroup)
        launch_lu_update<64, NB>(A, lda, n, ks, ks + NB, kLuGroup - 1 - sp, Linv, LinvT, UinvT, m, s);
      else
        launch_lu_update<128, kLuGroup * NB>(A, lda, n, k0, ks + NB, 0, Linv, LinvT, UinvT, m, s);
    }
  }
factored:
  timer_end(m, FPDE_STAGE_LU, t, s);
  FPDE_HIP(hipGetLastError());
  return FPDE_OK;
}

// u = U^{-1} L^{-1} b from an existing factor; the inverses of its diagonal
// blocks are formed first (one workgroup per block).
int lu_solve(fpde_mesh *m, const double *LU, int64_t lda, int64_t n, const double *b, double *u, double *xs,
             hipStream_t s) {
  if (n == 0) return FPDE_OK;
  double *Linv, *LinvT, *UinvT;
  FPDE_TRY(lu_inverses(m, n, &Linv, &LinvT, &UinvT));
  const int nblk = (int)((n + NB - 1) / NB);
  FPDE_TRY(ensure_trsv_sync(m));
  int *tickets = m->tsync;
  const long t = timer_begin(m, s, FPDE_STAGE_TRSV);
  k_lu_inverses<<<nblk, 256, 0, s>>>(LU, lda, n, LinvT, UinvT);
  FPDE_TRY(trsv_begin(tickets, xs, 0, n, 1, u != b ? b : nullptr, u, 0, s));
  k_trsv_rows<double, false><<<nblk, 256, 0, s>>>(LU, lda, n, nblk, LinvT, u, xs, tickets, m->flag, BatchStrides{});
  k_trsv_rows<double, true><<<nblk, 256, 0, s>>>(LU, lda, n, nblk, UinvT, xs, u, tickets + 1, m->flag,
                                                 BatchStrides{});
  timer_end(m, FPDE_STAGE_TRSV, t, s);
  FPDE_HIP(hipGetLastError());
  return FPDE_OK;
}

}  // namespace fpde

using namespace fpde;

extern "C" int fpde_lu_factor(fpde_mesh *m, double *A, int64_t lda, int64_t *failed_pivot, void *stream) {
  if (!m || !A || lda < m->ndof) return FPDE_EINVAL;
  if (failed_pivot) *failed_pivot = -1;
  hipStream_t s = S(stream);
  const int64_t n = m->ndof;
  if (n == 0) return FPDE_OK;
  FPDE_TRY(lu_factor(m, A, lda, n, s));
  int64_t col = -1;
  const int f = take_flag(m, s, &col);
  if (f != 0) {
    if (failed_pivot) *failed_pivot = col;
    return f < 0 ? f : FPDE_EHIP;
  }
  return FPDE_OK;
}

extern "C" int fpde_lu_solve(fpde_mesh *m, const double *LU, int64_t lda, const double *b, double *u,
                             void *stream) {
  if (!m || !LU || !b || !u || lda < m->ndof) return FPDE_EINVAL;
  hipStream_t s = S(stream);
  const int64_t n = m->ndof;
  if (n == 0) return FPDE_OK;
  double *xs = nullptr;
  FPDE_TRY(dalloc(&xs, (size_t)n));
  int st = lu_solve(m, LU, lda, n, b, u, xs, s);
  const int f = take_flag(m, s);
  dfree(xs);
  if (st != FPDE_OK) return st;
  return f < 0 ? f : (f > 0 ? FPDE_EHIP : FPDE_OK);
}
