// Integration-path walk (Sec. 2.2) and the closed-form order-gamma
// Riemann-Liouville derivatives of the P1 basis functions (Sec. 2.1).
//
// The walk depends on the mesh and the rule only: it runs when a plan is built
// and leaves its segments there; the values of every order are then computed
// from the segments (k_values).
//
// One thread owns one half-ray (Gauss point x_g, direction s e_i).  Threads
// are numbered direction-major, h = dir * G + g, so a wavefront walks 64
// neighbouring Gauss points (Morton-ordered elements) in the same direction:
// similar path lengths, and the element records they touch overlap in L2.
//
// Per element E on the path, with u0 = x_g fixed for the whole walk:
//   b~ = (A^{-1}(u0 - v0), 1 - e^T A^{-1}(u0 - v0)),  d~ = (s A^{-1} e_i, -e^T s A^{-1} e_i)
//   r_max = min_{d~_j < 0} -b~_j / d~_j          (eq:cond)
//   k~_max = b~ + r_max d~                          (equ:ac)
// and the zero pattern of k~_max names the go-out m-face (Fig. 2): one zero
// -> the element across that face; more -> an element sharing the edge or
// vertex in which the ray advances (smallest id); none -> boundary reached.
// The arithmetic of the walk is IEEE FP64 without FMA contraction, in the
// same operation order as the reference definition, so element ids are
// reproducible bit for bit.
//
// On the segment [r_{k-1}, r_k] of element E_k the basis function of local
// vertex j has slope sigma = d psi / d x_i = (grad k_j)_i, and contributes
//   -s sigma (r_k^{1-gamma} - r_{k-1}^{1-gamma}) / Gamma(2 - gamma)
// to the side-s derivative at x_g (integration by parts of eq. def, m = 1;
// interior basis functions vanish at the path end, so no end-point term).
// A 4-slot window holds the current element's vertices; a vertex that leaves
// the window is emitted as one (dof, value) entry, so a vector has about
// (segments + 3) entries.
#include <hipcub/hipcub.hpp>

#include <cmath>

#include "fpde_internal.h"

namespace fpde {

enum WalkMode { W_COUNT = 0, W_STRUCT = 1 };

struct WalkArgs {
  const TetRec *rec;
  const double *xyz;
  const int32_t *tet;
  const int32_t *vt_off;
  const int32_t *vt_tet;
  int32_t *flag;
  int64_t *flag_aux;
  int64_t G;
  int64_t h0, n;   // half-rays [h0, h0 + n)
  int cap;         // max elements per half-ray
  int nq;
  const double *qbary;  // device: nq x 4 barycentric coordinates of the rule
  // W_COUNT
  int32_t *cnt;    // n: entries per half-ray
  int32_t *len;    // n or null: elements per path
  uint64_t *hash;  // n or null
  int32_t *ids;    // n*cap or null
  double *rend;    // n*cap or null
  // W_STRUCT
  const int64_t *off, *soff;  // first entry and segment of half-ray h (global)
  int32_t *ent_dof;
  SegRec *seg;
};

struct Isect {
  double bt[4], dt[4];
  double r_max;
  int jexit;  // coordinate whose ratio set r_max (first one on ties)
};

// entry (r, i) of A^{-1} with a lane-varying axis i, without indexing the
// record dynamically (which would spill it to scratch)
__device__ __forceinline__ double Mcol(const TetRec &R, int r, int i) {
  const double a = R.M[3 * r], b = R.M[3 * r + 1], c = R.M[3 * r + 2];
  return i == 0 ? a : (i == 1 ? b : c);
}

__device__ __forceinline__ void isect(const TetRec &R, const double *u0, int i, int s, Isect &o) {
  const double b0 = u0[0] - R.v0[0];
  const double b1 = u0[1] - R.v0[1];
  const double b2 = u0[2] - R.v0[2];
#pragma unroll
  for (int r = 0; r < 3; r++) {
    o.bt[r + 1] = (R.M[3 * r + 0] * b0 + R.M[3 * r + 1] * b1) + R.M[3 * r + 2] * b2;
    const double m = Mcol(R, r, i);
    o.dt[r + 1] = (s > 0) ? m : -m;
  }
  o.bt[0] = 1.0 - ((o.bt[1] + o.bt[2]) + o.bt[3]);
  o.dt[0] = -((o.dt[1] + o.dt[2]) + o.dt[3]);
  double rm = INFINITY;
  int je = -1;
#pragma unroll
  for (int j = 0; j < 4; j++) {
    if (o.dt[j] < 0.0) {
      const double r = -o.bt[j] / o.dt[j];
      if (r < rm) {
        rm = r;
        je = j;
      }
    }
  }
  o.r_max = rm;
  o.jexit = je;
}

__device__ __forceinline__ TetRec load_rec(const TetRec *rec, int64_t t) {
  TetRec R;
  const double4 *p = reinterpret_cast<const double4 *>(rec + t);
  double4 a = p[0], b = p[1], c = p[2], d = p[3];
  R.M[0] = a.x; R.M[1] = a.y; R.M[2] = a.z; R.M[3] = a.w;
  R.M[4] = b.x; R.M[5] = b.y; R.M[6] = b.z; R.M[7] = b.w;
  R.M[8] = c.x; R.v0[0] = c.y; R.v0[1] = c.z; R.v0[2] = c.w;
  const int4 *q = reinterpret_cast<const int4 *>(&d);
  int4 n = q[0], f = q[1];
  R.nbr[0] = n.x; R.nbr[1] = n.y; R.nbr[2] = n.z; R.nbr[3] = n.w;
  R.dof[0] = f.x; R.dof[1] = f.y; R.dof[2] = f.z; R.dof[3] = f.w;
  return R;
}

// Per-thread staging of a half-ray's consecutive outputs.  A thread writes
// its entries one at a time as the walk proceeds, and its neighbours in the
// wavefront write other half-rays' ranges, so plain stores leave every
// 64-byte segment of the output partly written for many steps (the caches
// evict such segments and the memory takes several partial writes per
// segment).  Instead each output goes to LDS slot (index mod L) of the
// thread's column, and an aligned run of L outputs leaves as 16-byte stores
// once its last element is known; the first and last runs of a half-ray,
// which it shares with its neighbours, are written element by element.
// The destination arrays are 256-byte aligned (device allocations).
template <class T, int L>
__device__ __forceinline__ void stage_put(T (*st)[256], T *__restrict__ out, int64_t base, int64_t e, T v) {
  static_assert(L * sizeof(T) == 64, "runs are 64-byte segments");
  const int tid = threadIdx.x;
  const int sl = (int)(e & (L - 1));
  st[sl][tid] = v;
  if (sl != L - 1) return;
  const int64_t c0 = e - (L - 1);
  if (c0 >= base) {
    if constexpr (sizeof(T) == 16) {
#pragma unroll
      for (int u = 0; u < L; u++) out[c0 + u] = st[u][tid];
    } else {
      int4 *p = reinterpret_cast<int4 *>(out + c0);
#pragma unroll
      for (int u = 0; u < L / 4; u++)
        p[u] = make_int4(st[4 * u][tid], st[4 * u + 1][tid], st[4 * u + 2][tid], st[4 * u + 3][tid]);
    }
  } else {
    for (int64_t q = base; q <= e; q++) out[q] = st[q & (L - 1)][tid];
  }
}

// the outputs of the last, incomplete run [max(base, end rounded down), end)
template <class T, int L>
__device__ __forceinline__ void stage_flush(T (*st)[256], T *__restrict__ out, int64_t base, int64_t end) {
  const int64_t c0 = end & ~(int64_t)(L - 1);
  for (int64_t q = c0 > base ? c0 : base; q < end; q++) out[q] = st[q & (L - 1)][threadIdx.x];
}

template <int MODE>
__global__ void __launch_bounds__(256) k_walk(WalkArgs a) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= a.n) return;
  const int64_t h = a.h0 + k;
  const int dir = (int)(h / a.G);
  const int64_t g = h - (int64_t)dir * a.G;
  const int i = dir >> 1, side = dir & 1;
  const int s = side ? 1 : -1;
  const int nq = a.nq;
  const int64_t t0 = g / nq;
  const int q = (int)(g - t0 * nq);

  // Gauss point x_g = sum_j beta_qj v_j, summed in vertex order
  double u0[3];
  {
    int32_t vv[4];
#pragma unroll
    for (int j = 0; j < 4; j++) vv[j] = a.tet[4 * t0 + j];
#pragma unroll
    for (int d = 0; d < 3; d++) {
      double acc = 0.0;
#pragma unroll
      for (int j = 0; j < 4; j++) acc = acc + a.qbary[4 * q + j] * a.xyz[3 * (int64_t)vv[j] + d];
      u0[d] = acc;
    }
  }

  // window of the current element's vertices (unknowns, -1 on the boundary) and
  // the slots they stand in
  int32_t wd[4] = {-1, -1, -1, -1};
  int ws[4] = {0, 0, 0, 0};
  int64_t nemit = 0;
  int64_t base = 0, sbase = 0;
  if (MODE == W_STRUCT) {
    base = a.off[h];
    sbase = a.soff[h];
  }
  SegRec sr{};  // the last segment, written once it is known which vertices end there

  // staging runs of the structure pass (node ids and segments)
  __shared__ int32_t st_dof[MODE == W_STRUCT ? 16 : 1][256];
  __shared__ SegRec st_seg[MODE == W_STRUCT ? 4 : 1][256];
  auto emit = [&](int32_t d) {
    if constexpr (MODE == W_STRUCT) stage_put<int32_t, 16>(st_dof, a.ent_dof, base, base + nemit, d);
    nemit++;
  };

  uint64_t hsh = 14695981039346656037ull;
  int64_t t = t0;
  double r_cur = 0.0;
  int nseg = 0;
  int status = FPDE_EPATH;  // cleared when the walk reaches the boundary
  for (int step = 0; step < a.cap + 64; step++) {
    const TetRec R = load_rec(a.rec, t);
    Isect o;
    isect(R, u0, i, s, o);
    if (!(o.r_max < INFINITY)) {
      status = FPDE_EPATH;
      break;
    }
    if (o.r_max > r_cur) {
      // segment [r_cur, r_max] in element t
      if (nseg >= a.cap) {
        status = FPDE_EPATH;
        break;
      }
      if (MODE == W_COUNT) {
        const uint32_t uid = (uint32_t)t;
#pragma unroll
        for (int b = 0; b < 4; b++) {
          hsh ^= (uint64_t)((uid >> (8 * b)) & 0xffu);
          hsh *= 1099511628211ull;
        }
        if (a.ids) a.ids[k * a.cap + nseg] = (int32_t)t;
        if (a.rend) a.rend[k * a.cap + nseg] = o.r_max;
      }
      // move the window onto this element's vertices
      {
        const int32_t nd[4] = {R.dof[0], R.dof[1], R.dof[2], R.dof[3]};
        int ns[4] = {-1, -1, -1, -1};
        int used = 0;
#pragma unroll
        for (int j = 0; j < 4; j++) {
          if (wd[j] < 0) continue;
          bool kept = false;
#pragma unroll
          for (int m = 0; m < 4; m++) {
            if (nd[m] == wd[j]) {
              ns[m] = ws[j];
              used |= 1 << ws[j];
              kept = true;
            }
          }
          if (!kept) {
            emit(wd[j]);
            if (MODE == W_STRUCT) sr.code |= 256u << j;
          }
        }
        if (MODE == W_STRUCT) {
          if (nseg > 0) stage_put<SegRec, 4>(st_seg, a.seg, sbase, sbase + nseg - 1, sr);
          sr.r = nseg > 0 ? o.r_max : -o.r_max;
          sr.tet = (int32_t)t;
          sr.code = 0;
#pragma unroll
          for (int m = 0; m < 4; m++) {
            if (ns[m] < 0) {  // a new vertex takes the first free slot
              ns[m] = __builtin_ctz(~used);
              used |= 1 << ns[m];
              sr.code |= 4096u << ns[m];
            }
            sr.code |= (uint32_t)ns[m] << (2 * m);
            ws[m] = ns[m];
          }
        }
#pragma unroll
        for (int j = 0; j < 4; j++) wd[j] = nd[j];
      }
      nseg++;
      r_cur = o.r_max;
    }
    // zero pattern of the volume coordinates at the go-out point: |k_j| is
    // compared with 1e-12 times the size of the two terms it is the
    // difference of (at least 1e-12); the coordinate that set r_max is zero
    // by construction
    int zmask = 0, nz = 0, zf = -1;
#pragma unroll
    for (int j = 0; j < 4; j++) {
      const double p = o.r_max * o.dt[j];
      const double kj = o.bt[j] + p;
      double sc = fabs(o.bt[j]);
      sc = fabs(p) > sc ? fabs(p) : sc;
      sc = sc < 1.0 ? 1.0 : sc;
      if (j == o.jexit || fabs(kj) <= 1e-12 * sc) {
        zmask |= 1 << j;
        nz++;
        zf = j;
      }
    }
    if (nz == 0 || nz == 4) {
      status = FPDE_EPATH;
      break;
    }
    if (nz == 1) {
      const int32_t nx = zf == 0 ? R.nbr[0] : (zf == 1 ? R.nbr[1] : (zf == 2 ? R.nbr[2] : R.nbr[3]));
      if (nx < 0) {  // boundary reached
        status = 0;
        break;
      }
      t = nx;
      continue;
    }
    // edge or vertex: elements containing every vertex whose k != 0
    int32_t tv[4];
#pragma unroll
    for (int j = 0; j < 4; j++) tv[j] = a.tet[4 * t + j];
    const int first = __builtin_ctz((~zmask) & 0xf);  // nz <= 3, so one vertex is kept
    const int32_t v_first = (first == 0) ? tv[0] : (first == 1) ? tv[1] : (first == 2) ? tv[2] : tv[3];
    int64_t best = -1;
    for (int32_t p = a.vt_off[v_first]; p < a.vt_off[v_first + 1]; p++) {
      const int64_t c = a.vt_tet[p];
      if (c == t) continue;
      int32_t cv[4];
#pragma unroll
      for (int j = 0; j < 4; j++) cv[j] = a.tet[4 * c + j];
      bool all = true;
#pragma unroll
      for (int m = 0; m < 4; m++) {
        if ((zmask >> m) & 1) continue;
        const bool f = (cv[0] == tv[m]) || (cv[1] == tv[m]) || (cv[2] == tv[m]) || (cv[3] == tv[m]);
        all = all && f;
      }
      if (!all) continue;
      const TetRec Rc = load_rec(a.rec, c);
      Isect oc;
      isect(Rc, u0, i, s, oc);
      if (oc.r_max - r_cur > 1e-12 * r_cur) {
        best = c;
        break;
      }
    }
    if (best < 0) {  // boundary reached through an edge or vertex
      status = 0;
      break;
    }
    t = best;
  }
  if (status == 0 && nseg == 0) status = FPDE_EPATH;
  if (status != 0) {
    set_flag(a.flag, status);
    atomicCAS((unsigned long long *)a.flag_aux, ~0ull, (unsigned long long)h);
    if (MODE == W_COUNT) a.cnt[k] = 0;
    return;
  }
  // flush the last element's vertices
#pragma unroll
  for (int j = 0; j < 4; j++)
    if (wd[j] >= 0) {
      emit(wd[j]);
      if (MODE == W_STRUCT) sr.code |= 256u << j;
    }
  if constexpr (MODE == W_STRUCT) {
    stage_put<SegRec, 4>(st_seg, a.seg, sbase, sbase + nseg - 1, sr);
    stage_flush<int32_t, 16>(st_dof, a.ent_dof, base, base + nemit);
    stage_flush<SegRec, 4>(st_seg, a.seg, sbase, sbase + nseg);
  }
  if (MODE == W_COUNT) {
    a.cnt[k] = (int32_t)nemit;
    if (a.len) a.len[k] = nseg;
    if (a.hash) a.hash[k] = hsh;
  }
}

// ---- Values from the segments ----
//
// A wavefront takes the segments of kStripRays half-rays of one direction, kStep
// at a time, one per lane: the power at the segment's end (the one at its start
// comes from the lane below), and the contribution of each of the element's
// vertices to LDS, in the row of the slot that the vertex stands in while it
// stays in the window.  An entry is then the sum of a run of its slot's row, one
// lane per entry, in path order, and the entries leave coalesced.  What a run
// has summed up by the end of the step is carried in front of the row.
//
// Bound by instruction issue (some 350 per step), at 2.1 of the 4.7 TB/s of a
// copy (16 bytes read per segment, 8 written per entry).  (Walking again for every order, one thread per
// half-ray, was bound by the intersections, three divisions each, and by lanes
// waiting for the longest path of their wavefront: 0.76 against 0.30 ms for
// 216 392 points, 9.2 against 4.6 ms for 1 670 977.)
constexpr int kStripRays = 16;

struct ValArgs {
  const SegRec *seg;
  const int64_t *strip;  // first segment of each strip, strips_per_dir per direction
  const int64_t *off;
  const double4 *slope;  // [axis][element]: slopes of the four volume coordinates
  int64_t G, nt, strips_per_dir;
  int64_t strip0, n_strip;
  // per axis: 1 - gamma_i, 1/Gamma(2 - gamma_i); psi(2 - gamma)/2 (one order)
  double e[3], inv_g2[3], half_psi0;
  double *ent_val;
  const double2 *grad;  // adjoint: [axis][element] derivatives of u and lam
  double *adj;          // adjoint: 4 per half-ray
};

// slopes of the volume coordinates along the axes
__global__ void k_slopes(const TetRec *__restrict__ rec, int64_t nt, double4 *__restrict__ slope) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= nt) return;
  const TetRec R = load_rec(rec, t);
#pragma unroll
  for (int i = 0; i < 3; i++) {
    const double a = R.M[i], b = R.M[3 + i], c = R.M[6 + i];
    slope[i * nt + t] = make_double4(-((a + b) + c), a, b, c);
  }
}

__global__ void k_strip_starts(const int64_t *__restrict__ soff, int64_t G, int64_t per_dir, int64_t n,
                               int64_t n_half, int64_t *__restrict__ strip) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k > n) return;
  strip[k] = soff[k == n ? n_half : (k / per_dir) * G + (k % per_dir) * kStripRays];
}

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ int below(uint64_t m) {  // bits of m below this lane's
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

__device__ __forceinline__ SegRec load_seg(const SegRec *p) {
  const int4 v = *reinterpret_cast<const int4 *>(p);
  SegRec r;
  r.r = __hiloint2double(v.y, v.x);
  r.tet = v.z;
  r.code = (uint32_t)v.w;
  return r;
}

// r^e = 2^(e log2 r) for normal r > 0 and e in [0, 1], and log2 r.  With
// m = r 2^-k in [1/sqrt 2, sqrt 2): log2 m = (2 / ln 2) atanh(q), q = (m - 1) /
// (m + 1), |q| < 0.1716, the series up to q^19 (rest below 2^-57 of it); k +
// log2 m and its product with e are kept as unevaluated sums of two doubles, and
// 2^f on [-1/2, 1/2] is its series up to f^13 (rest below 2^-57).  At most 1.8
// units of 2^-53 off over r in [1e-8, 1e4], where exp(e log(r)) has 4 to 32, in
// a third of its instructions: the coefficients stand in scalar registers.
__constant__ double kAtanh[10] = {0x1.71547652b82fep+1, 0x1.ec709dc3a03fdp-1, 0x1.2776c50ef9bfep-1,
                                  0x1.a61762a7aded9p-2, 0x1.484b13d7c02a9p-2, 0x1.0c9a84994022dp-2,
                                  0x1.c68f568d3176p-3,  0x1.89f3b1694cffep-3, 0x1.5b9ac9b743f0dp-3,
                                  0x1.3703c1f4d0ffep-3};  // 2 / ((2 n + 1) ln 2)
__constant__ double kExp2[14] = {0x1p+0,                0x1.62e42fefa39efp-1,  0x1.ebfbdff82c58fp-3,
                                 0x1.c6b08d704a0cp-5,   0x1.3b2ab6fba4e77p-7,  0x1.5d87fe78a6731p-10,
                                 0x1.430912f86c787p-13, 0x1.ffcbfc588b0c7p-17, 0x1.62c0223a5c824p-20,
                                 0x1.b5253d395e7c4p-24, 0x1.e4cf5158b8ecap-28, 0x1.e8cac7351bb25p-32,
                                 0x1.c3bd650fc2986p-36, 0x1.816193166d0f9p-40};  // ln 2^n / n!
__device__ __forceinline__ double pow_unit(double r, double e, double *log2r = nullptr) {
  int k = __builtin_amdgcn_frexp_exp(r);
  double m = __builtin_amdgcn_frexp_mant(r);  // [1/2, 1)
  const bool low = m < 0.70710678118654752;
  m = low ? m + m : m;
  k = low ? k - 1 : k;
  const double f = m - 1.0, d = m + 1.0;
  double x = __builtin_amdgcn_rcp(d);
  x = fma(fma(-d, x, 1.0), x, x);
  x = fma(fma(-d, x, 1.0), x, x);
  double q = f * x;
  q = fma(fma(-d, q, f), x, q);
  const double z = q * q;
  double p = kAtanh[9];
#pragma unroll
  for (int n = 8; n >= 0; n--) p = fma(p, z, kAtanh[n]);
  const double t = p * q, kd = (double)k, hi = kd + t, lo = t - (hi - kd);
  if (log2r) *log2r = hi;
  const double y = e * hi, yl = fma(e, lo, fma(e, hi, -y));
  const double n = __builtin_rint(y), g = (y - n) + yl;
  double w = kExp2[13];
#pragma unroll
  for (int c = 12; c >= 0; c--) w = fma(w, g, kExp2[c]);
  return __builtin_amdgcn_ldexp(w, (int)n);
}

constexpr int kValWaves = 4;
// Segments per step of k_values: about as many entries end as segments are
// taken, and four lanes are wanted for the carried sums, so that 60 mostly leave
// one round of the entry loop (48 / 52 / 56 / 60 / 64: 0.35 / 0.33 / 0.31 / 0.30 /
// 0.31 ms for 216 392 points).
constexpr int kStep = 60;

__global__ void __launch_bounds__(64 * kValWaves) k_values(ValArgs a) {
  __shared__ double row_[kValWaves * 4 * 65 + 4];  // per wavefront [slot][0]: carried sum; [1 + lane]
  __shared__ uint16_t list_[kValWaves][4 * 64];   // entries of the step: slot, last lane
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t q = (int64_t)blockIdx.x * kValWaves + wave;
  if (q >= a.n_strip) return;
  double(*row)[65] = reinterpret_cast<double(*)[65]>(row_ + wave * 4 * 65);
  uint16_t *list = list_[wave];
  const int64_t strip = a.strip0 + q;
  const int dir = (int)(strip / a.strips_per_dir), i = dir >> 1;
  const int64_t h0 = dir * a.G + (strip - dir * a.strips_per_dir) * kStripRays;
  const double sgn = (dir & 1) ? -1.0 : 1.0;
  const double ei = a.e[i], gi = a.inv_g2[i];
  const double4 *slope = a.slope + i * a.nt;
  const int64_t s1 = a.strip[strip + 1];
  double *out = a.ent_val + a.off[h0];
  double P_last = 0.0;
  SegRec nx{};
  int64_t s = a.strip[strip];
  if (lane < kStep && s + lane < s1) nx = load_seg(a.seg + s + lane);
  for (; s < s1; s += kStep) {
    const SegRec sr = nx;  // lanes past the end: r = 0, nothing new, nothing emitted
    const bool act = lane < kStep && s + lane < s1;
    const double4 sl = slope[sr.tet];
    nx = SegRec{};
    if (lane < kStep && s + kStep + lane < s1) nx = load_seg(a.seg + s + kStep + lane);
    const double P_hi = act ? pow_unit(fabs(sr.r), ei) : 0.0;
    double P_lo = __shfl_up(P_hi, 1, 64);
    if (lane == 0) P_lo = P_last;
    if (sr.r < 0.0) P_lo = 0.0;  // the half-ray's first segment
    P_last = __shfl(P_hi, kStep - 1, 64);
    const double dP = gi * (P_hi - P_lo);
    row[sr.code & 3][1 + lane] = (sgn * sl.x) * dP;
    row[(sr.code >> 2) & 3][1 + lane] = (sgn * sl.y) * dP;
    row[(sr.code >> 4) & 3][1 + lane] = (sgn * sl.z) * dP;
    row[(sr.code >> 6) & 3][1 + lane] = (sgn * sl.w) * dP;
    // which slots get a new vertex, and the places of the entries that end
    const uint64_t new0 = __ballot(sr.code >> 12 & 1), new1 = __ballot(sr.code >> 13 & 1),
                   new2 = __ballot(sr.code >> 14 & 1), new3 = __ballot(sr.code >> 15 & 1);
    const uint32_t em = sr.code >> 8 & 15u;
    const uint32_t cnt = __popc(em);
    const uint64_t b0 = __ballot(cnt & 1), b1 = __ballot(cnt & 2), b2 = __ballot(cnt & 4);
    int pos = below(b0) + 2 * below(b1) + 4 * below(b2);
    const int total = __popcll(b0) + 2 * __popcll(b1) + 4 * __popcll(b2);
#pragma unroll
    for (int j = 0; j < 4; j++)
      if (em >> j & 1u) list[pos++] = (uint16_t)((sr.code >> (2 * j) & 3u) << 6 | lane);
    wave_sync();
    // one lane per entry, and one per slot for the sum to carry over
    double carry = 0.0;
    int cs = -1;
    for (int k = lane; k < total + 4; k += 64) {
      int slot, last;
      if (k < total) {
        slot = list[k] >> 6;
        last = list[k] & 63;
      } else {
        slot = cs = k - total;
        last = kStep - 1;
      }
      uint64_t m = slot < 2 ? (slot == 0 ? new0 : new1) : (slot == 2 ? new2 : new3);
      m &= ~0ull >> (63 - last);
      int x = m ? 64 - __clzll((long long)m) : 0;
      const double *c = &row[slot][x];  // up to four cells past the run are read and left out
      int left = last + 1 - x;          // cells after the first
      double v = *c;
      do {
        const double c1 = c[1], c2 = c[2], c3 = c[3], c4 = c[4];
        v += left > 0 ? c1 : 0.0;
        v += left > 1 ? c2 : 0.0;
        v += left > 2 ? c3 : 0.0;
        v += left > 3 ? c4 : 0.0;
        c += 4;
        left -= 4;
      } while (left > 0);
      if (k < total)
        out[k] = v;
      else
        carry = v;
    }
    wave_sync();
    if (cs >= 0) row[cs][0] = carry;
    out += total;
  }
}

// a.x b0 + .. + a.w b3 as if in twice the precision (compensated dot product by
// Ogita, Rump and Oishi): the terms cancel to the element's size over the
// domain's, and every ray through the element shares the result's rounding.
__device__ __forceinline__ double dot4_comp(const double4 &a, const double (&b)[4]) {
  const double c[4] = {a.x, a.y, a.z, a.w};
  double p = c[0] * b[0], e = fma(c[0], b[0], -p);
#pragma unroll
  for (int j = 1; j < 4; j++) {
    const double h = c[j] * b[j], l = fma(c[j], b[j], -h);
    const double t = p + h, z = t - p;
    e += ((p - (t - z)) + (h - z)) + l;
    p = t;
  }
  return p + e;
}

// derivatives of u and lam along the axes, per element
__global__ void k_elem_grad(const TetRec *__restrict__ rec, const double4 *__restrict__ slope, int64_t nt,
                            const double *__restrict__ u, const double *__restrict__ lam,
                            double2 *__restrict__ grad) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= nt) return;
  double uu[4], ll[4];
#pragma unroll
  for (int j = 0; j < 4; j++) {
    const int32_t d = rec[t].dof[j];
    uu[j] = d < 0 ? 0.0 : u[d];
    ll[j] = d < 0 ? 0.0 : lam[d];
  }
#pragma unroll
  for (int i = 0; i < 3; i++) {
    const double4 c = slope[i * nt + t];
    grad[i * nt + t] = make_double2(dot4_comp(c, uu), dot4_comp(c, ll));
  }
}

// Per half-ray value.u, value.lam and their derivatives in alpha: on a segment
// all of an element's vertices share the power's difference, so the sum over
// the entries is one over the segments with the element's derivative of u (of
// lam).  Strips as in k_values; each lane sums one of the four for one half-ray.
// (Walking again with a gather of u and lam per entry: 1.13 against 0.31 ms for
// 168 308 points.)
__global__ void __launch_bounds__(64 * kValWaves) k_adjoint_rays(ValArgs a) {
  __shared__ double row_[kValWaves][4][64];
  __shared__ int start_[kValWaves][kStripRays + 1];
  static_assert(4 * kStripRays == 64, "one lane per half-ray and sum");
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t q = (int64_t)blockIdx.x * kValWaves + wave;
  if (q >= a.n_strip) return;
  double(*row)[64] = row_[wave];
  int *start = start_[wave];
  const int64_t strip = a.strip0 + q;
  const int dir = (int)(strip / a.strips_per_dir), i = dir >> 1;
  const int64_t g0 = (strip - dir * a.strips_per_dir) * kStripRays, h0 = dir * a.G + g0;
  const double sgn = (dir & 1) ? -1.0 : 1.0;
  const double ei = a.e[i], gi = a.inv_g2[i];
  const double2 *grad = a.grad + i * a.nt;
  const int64_t s0 = a.strip[strip], s1 = a.strip[strip + 1];
  if (lane <= kStripRays) start[lane] = 0x7fffffff;
  wave_sync();
  const int ray = lane >> 2, which = lane & 3;
  double P_last = 0.0, Q_last = 0.0, acc = 0.0;
  int seen = 0;
  for (int64_t s = s0; s < s1; s += 64) {
    SegRec sr{};
    const bool act = s + lane < s1;
    if (act) sr = load_seg(a.seg + s + lane);
    const double2 gr = grad[sr.tet];
    double P_hi = 0.0, Q_hi = 0.0;
    if (act) {
      double l;
      P_hi = pow_unit(fabs(sr.r), ei, &l);
      Q_hi = (l * 0.69314718055994531) * P_hi;
    }
    double P_lo = __shfl_up(P_hi, 1, 64), Q_lo = __shfl_up(Q_hi, 1, 64);
    if (lane == 0) {
      P_lo = P_last;
      Q_lo = Q_last;
    }
    const bool first = sr.r < 0.0;
    if (first) P_lo = Q_lo = 0.0;
    P_last = __shfl(P_hi, 63, 64);
    Q_last = __shfl(Q_hi, 63, 64);
    const double dP = sgn * (gi * (P_hi - P_lo));
    const double dQ = sgn * (gi * (a.half_psi0 * (P_hi - P_lo) - 0.5 * (Q_hi - Q_lo)));
    row[0][lane] = dP * gr.x;
    row[1][lane] = dP * gr.y;
    row[2][lane] = dQ * gr.x;
    row[3][lane] = dQ * gr.y;
    const uint64_t fm = __ballot(first);
    if (first) start[seen + below(fm)] = (int)(s - s0) + lane;  // < kStripRays starts in all
    seen += __popcll(fm);
    wave_sync();
    const int rel = (int)(s - s0), n = (int)(s1 - s < 64 ? s1 - s : 64);
    int x = start[ray] - rel, e = start[ray + 1] - rel;
    x = x < 0 ? 0 : x;
    e = e < n ? e : n;
    for (; x < e; x++) acc += row[which][x];
    wave_sync();
  }
  if (g0 + ray < a.G) a.adj[4 * h0 + lane] = acc;
}

__global__ void k_i32_to_i64(const int32_t *__restrict__ a, int64_t n, int64_t *__restrict__ b) {
  int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n) b[k] = a[k];
}

static inline unsigned nblk(int64_t n, int b = 256) { return (unsigned)((n + b - 1) / b); }

static WalkArgs base_args(fpde_mesh *m, const Plan &P, const QuadRule &rule) {
  WalkArgs a{};
  a.rec = m->rec;
  a.xyz = m->xyz;
  a.tet = m->tet;
  a.vt_off = m->vt_off;
  a.vt_tet = m->vt_tet;
  a.flag = m->flag;
  a.flag_aux = m->flag_aux;
  a.G = P.G;
  a.cap = P.max_steps;
  a.nq = rule.nq;
  a.qbary = m->rules + rule_offset(rule.nq);
  return a;
}

template <int MODE>
static void launch_walk(const WalkArgs &a, hipStream_t s) {
  if (a.n <= 0) return;
  k_walk<MODE><<<nblk(a.n), 256, 0, s>>>(a);
}

void free_plan(Plan &P) {
  dfree(P.off); dfree(P.ent_dof); dfree(P.ent_val); dfree(P.ent_val2); dfree(P.adj);
  dfree(P.seg); dfree(P.strip);
  free_tubes(P.tubes);
  P = Plan();
}

// Tube cell edge of the accumulation, in mean element edges.  Narrower tubes
// have smaller node sets (blocks that fit the LDS whole, fuller 128-wide
// regions on the matrix cores) but more of them (block bytes and row places).
// Two assemblies, pass 1 and rows, at cells of 1.0 / 0.8 / 0.7 / 0.6 / 0.5:
// FP64 82 924 elements 5.5 / 4.9 / 4.9 / 5.0 / 5.2 ms, 19 672 elements (4
// points) 0.31 / 0.32 / 0.33 / 0.35 / 0.40 ms, mixed 151 907 elements
// 41.4 / 39.7 / 38.1 / 37.2 / 37.8 ms.
constexpr double kTubeCell = 0.7;

int plan_strips(Plan &P, const int64_t *soff, hipStream_t s) {
  P.strips = (P.G + kStripRays - 1) / kStripRays;
  const int64_t n = P.n_half / P.G * P.strips;
  FPDE_TRY(dalloc(&P.strip, n + 1));
  k_strip_starts<<<nblk(n + 1), 256, 0, s>>>(soff, P.G, P.strips, n, P.n_half, P.strip);
  return FPDE_OK;
}

static int build_plan(fpde_mesh *m, Plan &P, int nq, int max_steps, hipStream_t s) {
  QuadRule rule;
  FPDE_TRY(quad_rule(nq, &rule));
  P.nq = nq;
  P.max_steps = max_steps;
  P.G = m->nt * nq;
  P.n_half = 6 * P.G;
  int32_t *cnt = nullptr, *len = nullptr;
  int64_t *cnt64 = nullptr, *soff = nullptr;
  void *tmp = nullptr;
  int st = FPDE_OK;
  auto fail = [&](int code) {
    dfree(cnt); dfree(cnt64); dfree(len); dfree(soff);
    if (tmp) (void)hipFree(tmp);
    free_plan(P);
    return code;
  };
  if ((st = dalloc(&cnt, P.n_half + 1)) != FPDE_OK) return fail(st);
  if ((st = dalloc(&cnt64, P.n_half + 1)) != FPDE_OK) return fail(st);
  if ((st = dalloc(&P.off, P.n_half + 1)) != FPDE_OK) return fail(st);
  if ((st = dalloc(&len, P.n_half + 1)) != FPDE_OK) return fail(st);
  if ((st = dalloc(&soff, P.n_half + 1)) != FPDE_OK) return fail(st);
  if (hipMemsetAsync(cnt, 0, sizeof(int32_t) * (P.n_half + 1), s) != hipSuccess ||
      hipMemsetAsync(len, 0, sizeof(int32_t) * (P.n_half + 1), s) != hipSuccess)
    return fail(FPDE_EHIP);
  if (!m->slope) {  // for every plan of the mesh
    if ((st = dalloc(&m->slope, 3 * m->nt)) != FPDE_OK) return fail(st);
    k_slopes<<<nblk(m->nt), 256, 0, s>>>(m->rec, m->nt, m->slope);
  }

  WalkArgs a = base_args(m, P, rule);
  a.h0 = 0;
  a.n = P.n_half;
  a.cnt = cnt;
  a.len = len;
  launch_walk<W_COUNT>(a, s);
  k_i32_to_i64<<<nblk(P.n_half + 1), 256, 0, s>>>(cnt, P.n_half + 1, cnt64);
  size_t tb = 0;
  if (hipcub::DeviceScan::ExclusiveSum(nullptr, tb, cnt64, P.off, (int)(P.n_half + 1), s) != hipSuccess)
    return fail(FPDE_EHIP);
  if (hipMalloc(&tmp, tb) != hipSuccess) return fail(FPDE_ENOMEM);
  if (hipcub::DeviceScan::ExclusiveSum(tmp, tb, cnt64, P.off, (int)(P.n_half + 1), s) != hipSuccess)
    return fail(FPDE_EHIP);
  k_i32_to_i64<<<nblk(P.n_half + 1), 256, 0, s>>>(len, P.n_half + 1, cnt64);
  if (hipcub::DeviceScan::ExclusiveSum(tmp, tb, cnt64, soff, (int)(P.n_half + 1), s) != hipSuccess)
    return fail(FPDE_EHIP);
  if ((st = plan_strips(P, soff, s)) != FPDE_OK) return fail(st);
  int64_t n_seg = 0;
  if (hipMemcpyAsync(&n_seg, soff + P.n_half, sizeof(int64_t), hipMemcpyDeviceToHost, s) != hipSuccess)
    return fail(FPDE_EHIP);
  if (hipMemcpyAsync(&P.n_ent, P.off + P.n_half, sizeof(int64_t), hipMemcpyDeviceToHost, s) != hipSuccess)
    return fail(FPDE_EHIP);
  int f = take_flag(m, s);
  if (f != 0) return fail(f < 0 ? f : FPDE_EHIP);

  if (P.n_ent >= (int64_t(1) << 31)) return fail(FPDE_EUNSUPPORTED);  // 32-bit entry ids below
  if ((st = dalloc(&P.ent_dof, P.n_ent)) != FPDE_OK) return fail(st);
  if ((st = dalloc(&P.ent_val, P.n_ent)) != FPDE_OK) return fail(st);
  if ((st = dalloc(&P.seg, n_seg)) != FPDE_OK) return fail(st);
  a.off = P.off;
  a.soff = soff;
  a.ent_dof = P.ent_dof;
  a.seg = P.seg;
  launch_walk<W_STRUCT>(a, s);
  if (hipGetLastError() != hipSuccess) return fail(FPDE_EHIP);
  f = take_flag(m, s);
  if (f != 0) return fail(f < 0 ? f : FPDE_EHIP);
  dfree(cnt); dfree(cnt64); dfree(len); dfree(soff);
  (void)hipFree(tmp);
  tmp = nullptr;
  // sizes for reporting: entry pairs the accumulation multiplies
  {
    std::vector<int64_t> off(P.n_half + 1);
    if (hipMemcpy(off.data(), P.off, sizeof(int64_t) * (P.n_half + 1), hipMemcpyDeviceToHost) != hipSuccess)
      return fail(FPDE_EHIP);
    P.pairs = 0;
    P.max_ent = 0;
    for (int i = 0; i < 3; i++)
      for (int64_t g = 0; g < P.G; g++) {
        const int64_t hl = (int64_t)(2 * i) * P.G + g, hr = hl + P.G;
        const int64_t nl = off[hl + 1] - off[hl], nr = off[hr + 1] - off[hr];
        P.pairs += nl * nr;
        P.max_ent = std::max(P.max_ent, std::max(nl, nr));
      }
  }
  const TubeGeom q{3, m->nv, m->nt, m->xyz, m->tet, m->vol, m->rules + rule_offset(nq)};
  if ((st = build_tubes(m, P, q, kTubeCell, s)) != FPDE_OK) return fail(st);
  invalidate_values(&P);
  return FPDE_OK;
}

int plan_for(fpde_mesh *m, int nq, int max_steps, hipStream_t s, Plan **out) {
  if (nq != 4 && nq != 11) return FPDE_EINVAL;
  if (max_steps <= 0) max_steps = 4096;
  Plan &P = m->plan[nq == 4 ? 0 : 1];
  if (P.nq == nq && P.max_steps == max_steps) {
    *out = &P;
    return FPDE_OK;
  }
  free_plan(P);
  const long t = timer_begin(m, s, FPDE_STAGE_PLAN);
  FPDE_TRY(build_plan(m, P, nq, max_steps, s));
  timer_end(m, FPDE_STAGE_PLAN, t, s);
  *out = &P;
  return FPDE_OK;
}

static ValArgs val_args(const fpde_mesh *m, const Plan &P, int axis0, int axis1) {
  ValArgs a{};
  a.seg = P.seg;
  a.strip = P.strip;
  a.off = P.off;
  a.slope = m->slope;
  a.G = P.G;
  a.nt = m->nt;
  a.strips_per_dir = P.strips;
  a.strip0 = 2 * axis0 * P.strips;
  a.n_strip = 2 * (axis1 - axis0 + 1) * P.strips;
  return a;
}

// Fills the plan's entry values from its segments for the axes whose order
// changed, in one launch over the contiguous range of half-rays that covers
// them (the half-rays along e_i are dir = 2i, 2i + 1).
int ensure_values_axes(fpde_mesh *m, Plan *P, const double gamma[3], hipStream_t s, int slot) {
  double *cache = slot == 0 ? P->val_gamma : P->val_gamma2;
  if (slot == 1 && !P->ent_val2) FPDE_TRY(dalloc(&P->ent_val2, P->n_ent));
  double *dest = slot == 0 ? P->ent_val : P->ent_val2;
  int i0 = 3, i1 = -1;
  for (int i = 0; i < 3; i++)
    if (cache[i] != gamma[i]) {
      i0 = i < i0 ? i : i0;
      i1 = i;
    }
  if (i1 < 0) return FPDE_OK;
  ValArgs a = val_args(m, *P, i0, i1);
  for (int i = 0; i < 3; i++) {
    const Order o = gamma_scalars(gamma[i]);
    a.e[i] = o.e;
    a.inv_g2[i] = o.inv_g2;
  }
  a.ent_val = dest;
  const long t = timer_begin(m, s, FPDE_STAGE_WALK);
  k_values<<<nblk(a.n_strip, kValWaves), 64 * kValWaves, 0, s>>>(a);
  timer_end(m, FPDE_STAGE_WALK, t, s);
  if (hipGetLastError() != hipSuccess) {
    invalidate_values(P);
    return FPDE_EHIP;
  }
  for (int i = i0; i <= i1; i++) cache[i] = gamma[i];
  return FPDE_OK;
}

int ensure_values(fpde_mesh *m, Plan *P, double alpha, hipStream_t s) {
  const double g[3] = {0.5 * alpha, 0.5 * alpha, 0.5 * alpha};
  return ensure_values_axes(m, P, g, s);
}

// Adjoint dots per half-ray: value.u, value.lam, (d/dalpha value).u,
// (d/dalpha value).lam.
int walk_adjoint(fpde_mesh *m, Plan *P, double alpha, const double *u, const double *lam, hipStream_t s) {
  const Order o = order_scalars(alpha);
  if (!P->adj) FPDE_TRY(dalloc(&P->adj, 4 * P->n_half + 6 * m->nt));
  double2 *grad = (double2 *)(P->adj + 4 * P->n_half);
  ValArgs a = val_args(m, *P, 0, 2);
  for (int i = 0; i < 3; i++) {
    a.e[i] = o.e;
    a.inv_g2[i] = o.inv_g2;
  }
  a.half_psi0 = o.half_psi0;
  a.grad = grad;
  a.adj = P->adj;
  const long t = timer_begin(m, s, FPDE_STAGE_ADJOINT);
  k_elem_grad<<<nblk(m->nt), 256, 0, s>>>(m->rec, m->slope, m->nt, u, lam, grad);
  k_adjoint_rays<<<nblk(a.n_strip, kValWaves), 64 * kValWaves, 0, s>>>(a);
  timer_end(m, FPDE_STAGE_ADJOINT, t, s);
  FPDE_HIP(hipGetLastError());
  return FPDE_OK;
}

}  // namespace fpde

using namespace fpde;

extern "C" int fpde_plan(fpde_mesh *m, int quad_points, int max_steps, void *stream) {
  if (!m) return FPDE_EINVAL;
  Plan *P = nullptr;
  return plan_for(m, quad_points, max_steps, S(stream), &P);
}

extern "C" int fpde_paths(fpde_mesh *m, int quad_points, int dir, int64_t g0, int64_t count, int max_steps,
                          int32_t *len, uint64_t *hash, int32_t *ids, double *rend, void *stream) {
  if (!m || dir < 0 || dir > 5 || g0 < 0 || count < 0 || !len || !hash) return FPDE_EINVAL;
  QuadRule rule;
  FPDE_TRY(quad_rule(quad_points, &rule));
  if (max_steps <= 0) max_steps = 4096;
  const int64_t G = m->nt * quad_points;
  if (g0 + count > G) return FPDE_EINVAL;
  if (count == 0) return FPDE_OK;
  hipStream_t s = S(stream);
  Plan tmp;
  tmp.G = G;
  tmp.max_steps = max_steps;
  int32_t *cnt = nullptr;
  FPDE_TRY(dalloc(&cnt, count));
  WalkArgs a = base_args(m, tmp, rule);
  a.h0 = (int64_t)dir * G + g0;
  a.n = count;
  a.cnt = cnt;
  a.len = len;
  a.hash = hash;
  a.ids = ids;
  a.rend = rend;
  launch_walk<W_COUNT>(a, s);
  int f = (hipGetLastError() == hipSuccess) ? take_flag(m, s) : FPDE_EHIP;
  dfree(cnt);
  return f;
}

extern "C" int fpde_ray_values(fpde_mesh *m, int quad_points, double alpha, int dir, int64_t g0, int64_t count,
                               int64_t *off, int32_t *dof, double *val, int64_t capacity, void *stream) {
  if (!m || !off || dir < 0 || dir > 5 || g0 < 0 || count < 0) return FPDE_EINVAL;
  if (!(alpha > 1.0 && alpha <= 2.0)) return FPDE_EALPHA;
  hipStream_t s = S(stream);
  Plan *P = nullptr;
  FPDE_TRY(plan_for(m, quad_points, 0, s, &P));
  if (g0 + count > P->G) return FPDE_EINVAL;
  FPDE_TRY(ensure_values(m, P, alpha, s));
  const int64_t h0 = (int64_t)dir * P->G + g0;
  FPDE_HIP(hipMemcpyAsync(off, P->off + h0, sizeof(int64_t) * (count + 1), hipMemcpyDeviceToHost, s));
  FPDE_HIP(hipStreamSynchronize(s));
  const int64_t e0 = off[0];
  for (int64_t k = 0; k <= count; k++) off[k] -= e0;
  const int64_t n = off[count];
  int f = take_flag(m, s);
  if (f != 0) return f;
  if (n > capacity || (n > 0 && (!dof || !val))) return FPDE_EINVAL;
  if (n > 0) {
    FPDE_HIP(hipMemcpyAsync(dof, P->ent_dof + e0, sizeof(int32_t) * n, hipMemcpyDeviceToHost, s));
    FPDE_HIP(hipMemcpyAsync(val, P->ent_val + e0, sizeof(double) * n, hipMemcpyDeviceToHost, s));
    FPDE_HIP(hipStreamSynchronize(s));
  }
  return FPDE_OK;
}

extern "C" int fpde_plan_info(fpde_mesh *m, int quad_points, int64_t *out, void *stream) {
  if (!m || !out) return FPDE_EINVAL;
  Plan *P = nullptr;
  FPDE_TRY(plan_for(m, quad_points, 0, S(stream), &P));
  out[0] = P->n_half;
  out[1] = P->n_ent;
  out[2] = P->pairs;
  out[3] = P->max_ent;
  out[4] = P->tubes.n_tubes;
  out[5] = P->tubes.n_u;
  out[6] = P->tubes.max_u;
  out[7] = P->tubes.blk_n * (int64_t)sizeof(double);
  return FPDE_OK;
}
