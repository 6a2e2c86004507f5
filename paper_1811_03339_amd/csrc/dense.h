// Dense 64-wide building blocks shared by the Cholesky (SPD) and LU
// (non-symmetric) factorizations and their triangular solves: the tile
// product staged through LDS, wavefront helpers, and the block-row
// triangular solve with ticket ordering, whose entries are their own flags.
#pragma once

#include "fpde_internal.h"

namespace fpde {

constexpr int NB = 64;

// LDS written by some lanes of a wavefront and then read by other lanes of
// the same wavefront (the wavefront's LDS operations complete in order).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ double read_lane(double v, int l) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), l);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), l);
  return __hiloint2double(hi, lo);
}

// Forces v to be computed at this point of the program.
__device__ __forceinline__ void pin(double &v) { asm volatile("" : "+v"(v)); }

// Lane-dependent index whose comparisons the compiler must not hoist out of
// the enclosing loop (each hoisted comparison pins a 64-bit lane mask).
__device__ __forceinline__ int opaque(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// Staging of the 64 x 64 tile products P Q^T over a 64-deep inner dimension
// (P and Q given as row pointers with leading dimensions; rows past
// `prow`/`qrow` (>= 1) read as zero): 256 threads load rows lr + 8 it,
// column lc of a 32-deep chunk.  The second chunk's global loads are issued
// before the first chunk's arithmetic, and every load reads a valid address
// (rows clamped, then zeroed), so a thread's loads are all in flight
// together.
template <class T>
__device__ __forceinline__ void stage_load(const T *__restrict__ P, int64_t ldp, int prow, const T *__restrict__ Q,
                                           int64_t ldq, int qrow, int kk, int lr, int lc, T (&pr)[8], T (&qr)[8]) {
#pragma unroll
  for (int it = 0; it < 8; it++) {
    const int rr = lr + 8 * it;
    pr[it] = P[(int64_t)(rr < prow ? rr : prow - 1) * ldp + kk + lc];
    qr[it] = Q[(int64_t)(rr < qrow ? rr : qrow - 1) * ldq + kk + lc];
  }
}


typedef double f64x4 __attribute__((ext_vector_type(4)));

// acc += sP[rows][0..32) sQ[columns][0..32)^T for this wavefront's 32 x 32
// quarter (rows rm, rm + 16, columns cm, cm + 16 of the lane's 16-groups;
// kq = lane >> 4 picks the slice row of the 4-deep operands)
__device__ __forceinline__ void mfma_chunk(const double (*sP)[33], const double (*sQ)[33], int rm, int cm, int kq,
                                           f64x4 acc[2][2]) {
#pragma unroll
  for (int k4 = 0; k4 < 32; k4 += 4) {
    const double a0 = sP[rm][k4 + kq], a1 = sP[rm + 16][k4 + kq];
    const double b0 = sQ[cm][k4 + kq], b1 = sQ[cm + 16][k4 + kq];
    acc[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b0, acc[0][0], 0, 0, 0);
    acc[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b1, acc[0][1], 0, 0, 0);
    acc[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b0, acc[1][0], 0, 0, 0);
    acc[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b1, acc[1][1], 0, 0, 0);
  }
}

__device__ __forceinline__ void mfma_out(const f64x4 acc[2][2], double out[16]) {
#pragma unroll
  for (int a = 0; a < 2; a++)
#pragma unroll
    for (int b = 0; b < 2; b++)
#pragma unroll
      for (int i = 0; i < 4; i++) out[(2 * a + b) * 4 + i] = acc[a][b][i];
}

// The same 64 x 64 product on the matrix cores, FP64: wavefront w owns the
// 32 x 32 quarter (w >> 1, w & 1) as four 16 x 16 tiles, each accumulated
// by v_mfma_f64_16x16x4f64 over 4-deep slices of the inner dimension
// (A operand: lane l holds P[row l & 15][k + (l >> 4)]; B operand:
// Q[column l & 15][k + (l >> 4)]).  Result: out[(2 a + b) 4 + i] is tile
// (a, b) of the quarter at row 4 i + (l >> 4), column l & 15.
template <int KD = NB>
__device__ __forceinline__ void tile_nt_mfma(const double *__restrict__ P, int64_t ldp, int prow,
                                             const double *__restrict__ Q, int64_t ldq, int qrow, double (*sP)[33],
                                             double (*sQ)[33], double out[16]) {
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int lc = tid & 31, lr = tid >> 5;
  const int rm = 32 * (w >> 1) + (lane & 15), cm = 32 * (w & 1) + (lane & 15), kq = lane >> 4;
  f64x4 acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; a++)
#pragma unroll
    for (int b = 0; b < 2; b++) acc[a][b] = f64x4{0.0, 0.0, 0.0, 0.0};
  double pr[8], qr[8];
  stage_load<double>(P, ldp, prow, Q, ldq, qrow, 0, lr, lc, pr, qr);
#pragma unroll
  for (int kk = 0; kk < KD; kk += 32) {
#pragma unroll
    for (int it = 0; it < 8; it++) {
      const int rr = lr + 8 * it;
      sP[rr][lc] = rr < prow ? pr[it] : 0.0;
      sQ[rr][lc] = rr < qrow ? qr[it] : 0.0;
    }
    __syncthreads();
    if (kk + 32 < KD) stage_load<double>(P, ldp, prow, Q, ldq, qrow, kk + 32, lr, lc, pr, qr);
    mfma_chunk(sP, sQ, rm, cm, kq, acc);
    __syncthreads();
  }
  mfma_out(acc, out);
}

// 64 x 64 tile product over a KD-deep inner dimension (a multiple of 32)
// for the factorization kernels, on the matrix cores in FP64 and in FP32.  Value q of the 16 a thread holds sits at tile row
// frag_row<T>(q), column frag_col<T>(q).
template <int KD = NB>
__device__ __forceinline__ void tile_product(const double *__restrict__ P, int64_t ldp, int prow,
                                             const double *__restrict__ Q, int64_t ldq, int qrow, double (*sP)[33],
                                             double (*sQ)[33], double out[16]) {
  tile_nt_mfma<KD>(P, ldp, prow, Q, ldq, qrow, sP, sQ, out);
}

typedef float f32x4 __attribute__((ext_vector_type(4)));

// FP32 on the matrix cores (v_mfma_f32_16x16x4f32), same quarters and
// operand layout as the FP64 product; this instruction's result is blocked:
// lane l holds rows 4 (l >> 4) + i, column l & 15 of each 16 x 16 tile.
template <int KD = NB>
__device__ __forceinline__ void tile_product(const float *__restrict__ P, int64_t ldp, int prow,
                                             const float *__restrict__ Q, int64_t ldq, int qrow, float (*sP)[33],
                                             float (*sQ)[33], float out[16]) {
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int lc = tid & 31, lr = tid >> 5;
  const int rm = 32 * (w >> 1) + (lane & 15), cm = 32 * (w & 1) + (lane & 15), kq = lane >> 4;
  f32x4 acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; a++)
#pragma unroll
    for (int b = 0; b < 2; b++) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
  float pr[8], qr[8];
  stage_load<float>(P, ldp, prow, Q, ldq, qrow, 0, lr, lc, pr, qr);
#pragma unroll
  for (int kk = 0; kk < KD; kk += 32) {
#pragma unroll
    for (int it = 0; it < 8; it++) {
      const int rr = lr + 8 * it;
      sP[rr][lc] = rr < prow ? pr[it] : 0.f;
      sQ[rr][lc] = rr < qrow ? qr[it] : 0.f;
    }
    __syncthreads();
    if (kk + 32 < KD) stage_load<float>(P, ldp, prow, Q, ldq, qrow, kk + 32, lr, lc, pr, qr);
#pragma unroll
    for (int k4 = 0; k4 < 32; k4 += 4) {
      const float a0 = sP[rm][k4 + kq], a1 = sP[rm + 16][k4 + kq];
      const float b0 = sQ[cm][k4 + kq], b1 = sQ[cm + 16][k4 + kq];
      acc[0][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0, b0, acc[0][0], 0, 0, 0);
      acc[0][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0, b1, acc[0][1], 0, 0, 0);
      acc[1][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1, b0, acc[1][0], 0, 0, 0);
      acc[1][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1, b1, acc[1][1], 0, 0, 0);
    }
    __syncthreads();
  }
#pragma unroll
  for (int a = 0; a < 2; a++)
#pragma unroll
    for (int b = 0; b < 2; b++)
#pragma unroll
      for (int i = 0; i < 4; i++) out[(2 * a + b) * 4 + i] = acc[a][b][i];
}

template <class T>
__device__ __forceinline__ int frag_row(int q);
template <class T>
__device__ __forceinline__ int frag_col(int q);
template <>
__device__ __forceinline__ int frag_row<double>(int q) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  return 32 * (w >> 1) + 16 * (q >> 3) + 4 * (q & 3) + (lane >> 4);
}
template <>
__device__ __forceinline__ int frag_col<double>(int q) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  return 32 * (w & 1) + 16 * ((q >> 2) & 1) + (lane & 15);
}
template <>
__device__ __forceinline__ int frag_row<float>(int q) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  return 32 * (w >> 1) + 16 * (q >> 3) + 4 * (lane >> 4) + (q & 3);
}
template <>
__device__ __forceinline__ int frag_col<float>(int q) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  return 32 * (w & 1) + 16 * ((q >> 2) & 1) + (lane & 15);
}

// Element strides between the systems of a strided batch (grid.y = system):
// matrix, diagonal-block inverses, vectors, tickets.  All zero for a single
// system.
struct BatchStrides {
  int64_t a = 0, l = 0, v = 0, x = 0;  // v: right-hand side / solution, x: intermediate vector
  int t = 0;
};
constexpr int kMaxBatch = 16;

constexpr int64_t kSpinLimit = int64_t(1) << 22;

// The blocks of a vector that the workgroups of one triangular-solve launch
// publish to each other are stored and loaded with relaxed device-scope
// atomic accesses, which are coherent across the XCDs' L2 caches by
// themselves.  Every entry is its own flag: the vector holds kUnset before the
// launch, and a reader polls the entries that it needs until none is unset.
// (With a flag per block, a hop to the next block took a store, the wait for it,
// the flag's store, a poll and the load, and forward a reduction through LDS:
// forward and backward 0.27 ms at N = 3 069 and 1.25 ms at 13 780, now 0.17 and
// 0.78 ms.)  No fence is needed, so no L2 write-back or invalidation
// (which would also evict the cached factor).
constexpr unsigned long long kUnset = ~0ull;  // a NaN; a result with these bits is stored as another
__device__ __forceinline__ double unset_value() { return __longlong_as_double((long long)kUnset); }
__device__ __forceinline__ bool is_unset(double v) { return (unsigned long long)__double_as_longlong(v) == kUnset; }
__device__ __forceinline__ double ld_dev(const double *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_dev(double *p, double v) {
  __hip_atomic_store(p, is_unset(v) ? __longlong_as_double(0x7ff8000000000000ll) : v, __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}

// v (this lane's entry p, loaded before) once it is set in every live lane of
// the wavefront; false after kSpinLimit polls.
__device__ __forceinline__ bool wait_set(const double *p, bool live, double &v) {
  for (int64_t it = 0; __any(live && is_unset(v)); it++) {
    if (it > kSpinLimit) return false;
    if (it > 0) __builtin_amdgcn_s_sleep(1);
    v = ld_dev(p);
  }
  return true;
}

// a + b after the upper 32 (odd 16) lanes of a and the lower 32 (even 16) of b
// changed places: in the lower (even) lanes the sum of a over both halves, in
// the upper (odd) ones that of b.
__device__ __forceinline__ double swap32_add(double a, double b) {
  const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false);
  return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}
__device__ __forceinline__ double swap16_add(double a, double b) {
  const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(a), __double2loint(b), false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(a), __double2hiint(b), false, false);
  return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}
template <int ctrl>
__device__ __forceinline__ double dpp_f64(double v) {
  return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(v), ctrl, 0xf, 0xf, true),
                          __builtin_amdgcn_update_dpp(0, __double2loint(v), ctrl, 0xf, 0xf, true));
}

// Sixteen per-lane values a[q] -> sum over the wave's 64 lanes of a[q], left
// in every lane with (lane >> 2) & 15 == q (butterfly that halves the vector at
// each exchange; lane swaps and DPP moves, no LDS).
__device__ __forceinline__ double wave_sum16(const double (&a)[16]) {
  const int lane = threadIdx.x & 63;
  double b[8], c[4], d[2];
  const bool h3 = lane & 8, h2 = lane & 4;
#pragma unroll
  for (int k = 0; k < 8; k++) b[k] = swap32_add(a[k], a[k + 8]);
#pragma unroll
  for (int k = 0; k < 4; k++) c[k] = swap16_add(b[k], b[k + 4]);
#pragma unroll
  for (int k = 0; k < 2; k++)  // lane ^ 8: rotate the row by 8
    d[k] = (h3 ? c[k + 2] : c[k]) + dpp_f64<0x128>(h3 ? c[k] : c[k + 2]);
  // lane ^ 4: mirror the half-row, then each group of four
  double e = (h2 ? d[1] : d[0]) + dpp_f64<0x1b>(dpp_f64<0x141>(h2 ? d[0] : d[1]));
  e += dpp_f64<0x4e>(e);  // lane ^ 2
  e += dpp_f64<0xb1>(e);  // lane ^ 1
  return e;
}

// Block-row triangular solve in one launch:
//   x_b = D_b^{-1} (y_b - sum_{c in S(b)} A_bc x_c),
// S(b) = {c < b} (UP = false, block rows handed out top to bottom) or
// {c > b} (UP = true, bottom to top); DinvT holds (D_b^{-1})^T, 64 x 64
// row-major per block.  x holds kUnset on entry; the forward solve leaves it in
// y, where the backward solve that follows publishes its result.  Used for L
// (Cholesky forward; LU forward with the unit lower factor) and U (LU backward),
// all read by block rows, so the loads of A are whole 64-wide row segments.  Each workgroup takes the next
// block row from an atomic ticket, so it only waits for block rows whose
// tickets were taken before its own by workgroups that are already running.
// Wave w owns rows 16w..16w+15 of the block row; lane = column within
// block c.
template <class T, bool UP>
__global__ void __launch_bounds__(256) k_trsv_rows(const T *__restrict__ A, int64_t lda, int64_t n, int nblk,
                                                   const T *__restrict__ DinvT, double *__restrict__ y,
                                                   double *__restrict__ x, int *ticket, int32_t *err,
                                                   BatchStrides bs) {
  __shared__ int sb, ok;
  __shared__ double rhs[NB];
  __shared__ double red[4][NB];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  {
    const int64_t z = blockIdx.y;  // system z of a strided batch (its own tickets)
    A += z * bs.a;
    DinvT += z * bs.l;
    y += z * bs.v;
    x += z * bs.x;
    ticket += z * bs.t;
  }
  if (tid == 0) {
    sb = atomicAdd(ticket, 1);
    ok = 1;
  }
  __syncthreads();
  if (sb >= nblk) return;
  const int b = UP ? nblk - 1 - sb : sb;
  const int nc = UP ? nblk - 1 - b : b;  // blocks of S(b)
  const int c_first = UP ? nblk - 1 : 0, step = UP ? -1 : 1;
  const int64_t r0 = (int64_t)b * NB;
  const int nb = (int)((n - r0) < NB ? (n - r0) : NB);
  // D_b^{-1}[lane][16w + q], read before any wait
  double li[16];
#pragma unroll
  for (int q = 0; q < 16; q++) li[q] = (double)DinvT[(int64_t)b * NB * NB + (int64_t)(16 * w + q) * NB + lane];
  int64_t roff[16];  // rows past the matrix end repeat the last row; their sums are dropped
#pragma unroll
  for (int q = 0; q < 16; q++) {
    const int r = 16 * w + q;
    roff[q] = (r0 + (r < nb ? r : nb - 1)) * lda;
  }
  // column of block c read by this lane (only the last block can be
  // partial: its missing columns load a valid entry and multiply zero)
  auto col_of = [&](int c) {
    const int64_t cc = (int64_t)c * NB + lane;
    return cc < n ? cc : n - 1;
  };
  // this lane's row of the right-hand side, in the lanes that wave_sum16 leaves it to
  const int row = 16 * w + (lane >> 2);
  const double yv = (lane & 3) == 0 && row < nb ? y[r0 + row] : 0.0;
  double part[16];
  T cur[16];
#pragma unroll
  for (int q = 0; q < 16; q++) {
    part[q] = 0.0;
    cur[q] = (T)0;
  }
  double xn = 0.0;
  if (nc > 0) {
    const int64_t cc = col_of(c_first);
    xn = ld_dev(&x[cc]);
#pragma unroll
    for (int q = 0; q < 16; q++) cur[q] = A[roff[q] + cc];
  }
  bool good = true;
  for (int it = 0; it < nc; it++) {
    const int c = c_first + step * it;
    const int64_t cc = col_of(c);
    const bool live = (int64_t)c * NB + lane < n;
    double xv = xn;
    if (!wait_set(&x[cc], live, xv)) {
      good = false;
      break;
    }
    if (!live) xv = 0.0;
    const int64_t cn = col_of(it + 1 < nc ? c + step : c);
    xn = ld_dev(&x[cn]);  // the next block's, mostly unset for the block row next in line
    T nxt[16];
#pragma unroll
    for (int q = 0; q < 16; q++) nxt[q] = A[roff[q] + cn];
#pragma unroll
    for (int q = 0; q < 16; q++) {
      part[q] = fma((double)cur[q], xv, part[q]);
      cur[q] = nxt[q];
    }
  }
  if (!good && lane == 0) ok = 0;
  const double sum = wave_sum16(part);
  if ((lane & 3) == 0) rhs[row] = (row < nb) ? yv - sum : 0.0;
  __syncthreads();
  double s = 0.0, s2 = 0.0;
#pragma unroll
  for (int q = 0; q < 8; q++) {
    s = fma(li[q], rhs[16 * w + q], s);
    s2 = fma(li[q + 8], rhs[16 * w + q + 8], s2);
  }
  red[w][lane] = s + s2;
  __syncthreads();
  // the block of x, written (published) by wavefront 0
  if (tid < nb) st_dev(&x[r0 + tid], (red[0][tid] + red[1][tid]) + (red[2][tid] + red[3][tid]));
  if (!UP && tid < nb) y[r0 + tid] = unset_value();  // every wavefront has read its rows
  if (tid == 0 && !ok) set_flag(err, FPDE_EHIP);
}

// Host helpers (solve.hip).
// Device buffer of `sets` x ceil(n / 64) inverses of 64 x 64 diagonal blocks
// (elements of `elem` bytes), kept in the mesh handle and grown on demand.
int ensure_linv(fpde_mesh *m, int64_t n, size_t elem, int sets, void **out);
// Two tickets per system for the solves.
int ensure_trsv_sync(fpde_mesh *m, int count = 1);
// Before the forward solve: the tickets are zero, x + z sx (z < count) is unset
// and, b not null, u + z sv = b + z sv (one kernel: no memset node when a caller
// captures a graph).
int trsv_begin(int *tickets, double *x, int64_t sx, int64_t n, int count, const double *b, double *u, int64_t sv,
               hipStream_t s);

}  // namespace fpde
