// Conjugate gradients with their scalars on the device: the state, and the end of
// an iteration as the next product takes it.
#pragma once

#include "fpde_internal.h"

namespace fpde {

struct CgState {
  double rz[2];        // r.z of the even and of the odd iterations
  double be;           // r.z over the one before, of the running iteration
  double bn2, rr, rt;  // b.b; r.r; true residual squared
  int64_t end;         // number of the launch that ended the loop, INT64_MAX: it runs
  int32_t done;        // how: 1: converged or not a number, 2: not positive definite
  int32_t it;
};

// Launches are numbered: 2 it is iteration it's product, 2 it + 1 what follows it.
// One that decides the end leaves its own number; a launch has nothing to do when
// an earlier one has ended the loop.  So whether a wavefront reads the word before
// or after a decision of its own launch makes no difference, and every wavefront
// of the launch goes the same way.
__device__ __forceinline__ bool cg_over(const CgState *st, int64_t launch) { return st->end < launch; }

// The product of iteration `it` of the loop (st null: a plain product y = K x).
// x is the direction of the iteration before; the new one, z + be x, is taken on
// the fly and left in pn (not x: other rows still read it).
struct CgStep {
  CgState *st = nullptr;
  const double *z = nullptr;
  double *pn = nullptr;
  const double *part = nullptr;  // np pairs of sums r.r, r.z of the iteration before
  double *dot = nullptr;         // per workgroup of the row pass: its part of pn.y
  int np = 0, it = 0;
  double tol = 0.0;
};

// sum of part[0 .. n) (stride ld), n <= 1024, in every thread; 256 threads
__device__ __forceinline__ double sum_parts(const double *__restrict__ part, int n, int ld, double *red) {
  double s = 0.0;
  for (int k = threadIdx.x; k < n; k += 256) s += part[(int64_t)k * ld];
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  __syncthreads();  // red may still be read from the sum before
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  return (red[0] + red[1]) + (red[2] + red[3]);
}

// Whether the loop has ended: |r| / |b| <= tol after iteration it - 1; else be.
// In every thread of a workgroup of 256 (red: 4 doubles); the first workgroup
// leaves it in the state.
__device__ __forceinline__ bool cg_ended(const CgStep &c, double &be, double *red, bool first_block) {
  if (cg_over(c.st, 2 * (int64_t)c.it)) return true;
  be = 0.0;
  if (c.it == 0) return false;
  const int odd = (c.it - 1) & 1;
  const double rr = sum_parts(c.part, c.np, 2, red), rz = sum_parts(c.part + 1, c.np, 2, red);
  be = rz / c.st->rz[odd];
  const bool end = !(sqrt(rr) / sqrt(c.st->bn2) > c.tol);
  if (first_block && threadIdx.x == 0) {
    c.st->rr = rr;
    c.st->it = c.it;
    c.st->rz[odd ^ 1] = rz;
    c.st->be = be;
    if (end) {
      c.st->done = 1;
      c.st->end = 2 * (int64_t)c.it;
    }
  }
  return end;
}

// entry j of the iteration's direction
__device__ __forceinline__ double cg_entry(const CgStep &c, double be, const double *__restrict__ x, int64_t j) {
  return c.it > 0 ? fma(be, x[j], c.z[j]) : x[j];
}

}  // namespace fpde
