// Accumulation of the dense stiffness matrix by tubes (Sec. 2.1 assembly,
// Sec. 2.3 sparsity).
//
// Every Gauss point g and axis i contribute the rank-2 update
//   A += w_g K_i c_alpha (l r^T + r l^T)
// where l and r are the derivative vectors of the two half-rays of the
// chord through x_g parallel to e_i.  Chords of nearby Gauss points run
// through nearly the same elements, so the pairs (g, i) are grouped into
// tubes: axis i and the rectangular cell of the plane orthogonal to e_i that
// holds x_g.  A tube's chords touch a small node set U_T (the union of its
// half-rays' entries), and its whole contribution is a dense |U_T| x |U_T|
// block.
//
//   plan (once per mesh and rule, independent of alpha and K):
//     tubes, the sorted node list U_T of each tube, for every entry its slot
//     (position of its node in U_T), and for every row the (tube, slot)
//     places where that node appears;
//   pass 1: one workgroup per (tube, band) reads the tube's entries once and
//     adds every product l_p r_q into an LDS band of the block; the band goes
//     to a scratch block in HBM.  The block is symmetric, B = S + S^T with
//     S = sum w l r^T, so each product of S is added once, at (min, max), and
//     expanded as it is written: in the full square for |U_T| <= 141, the
//     packed upper triangle for |U_T| <= 200, else a few bands of rows of that
//     triangle; larger blocks, and those of few heavy tubes, go in bands of full
//     rows that take both products.  Two assemblies of 82 924 elements (4 points, chords of 44
//     entries, up to 240 nodes a tube) took 9.5 ms with one row entry per lane
//     and larger tubes in bands of full rows that took both products, and take
//     3.0 ms; of 19 672 elements (11 points, 25 entries) 1.96 and 0.64 ms;
//   pass 2: one workgroup per row of A sums that row's slices of the tube
//     blocks into an LDS row and writes the row once.
// Each entry is read once per band of its tube (not once per node of its
// partner half-ray), and A is written once, without global atomics.
#include <hipcub/hipcub.hpp>

#include <algorithm>
#include <climits>
#include <cmath>
#include <vector>

#include "cg.h"
#include "fpde_internal.h"

namespace fpde {

namespace {

constexpr int kHash = 2 * kMaxTube;  // LDS hash slots per tube (int32 keys)
static_assert(kHash == 1 << 13, "hash_slot");
// Pass 1: LDS doubles of a band (157.5 KB: the packed triangle of |U_T| <= 200)
// and threads of its workgroup, one per CU.  The pass waits on its entry loads,
// so what counts is wavefronts per band: bands of 79 KB, two workgroups of 512
// threads per CU, took 6.2 ms against 5.1 ms on 82 924 elements (4 points),
// 0.85 ms against 0.81 ms on 19 672 (11 points), two assemblies each.
constexpr int kBand = 20160;
constexpr int kAccumThreads = 1024;
// Work items of the two pass-1 kernels.  A block goes in bands of the triangle (each
// product once, but every band meets all of them) up to kTriBands bands, and in
// bands of full rows (both products, but a band collects its own rows first) beyond,
// or when its tube has more of the whole work than one of kShares CUs: then in as
// many bands as it has shares, of at least kMinRows rows.  A tube's work is taken as
// pairs x nodes^2; tubes of kSplitFrom nodes are too little to split.
// Triangle against rows, one assembly: many tubes of 312 nodes (64 000 cubes, 3
// bands) 29.7 / 30.8 ms, 408 (52 x 24 x 24 cubes, 5 bands) 10.0 / 10.6 ms; few of 792
// (100 x 8 x 8) 6.2 / 4.1 ms, 1 596 (3 x 3 x 400) 64 / 12.8 ms.  Bars of 3 x 3 x 60 /
// 150 cells: one item per band 0.59 / 4.5 ms, with the shares 0.28 / 1.30 ms (kShares
// 128 / 512: 1.47 / 1.57 ms); general form 1.7 / 54 ms, now 0.35 / 1.8 ms.
constexpr int kShares = 256, kMinRows = 8, kSplitFrom = 64;
constexpr int64_t kTriBands = 5;

// row stride of a band in LDS: odd, so the rows of one column fall in distinct bank pairs
__host__ __device__ inline int band_stride(int U) { return U | 1; }

// rows [r0, r0 + R) of the row-packed upper triangle of a U x U block that fit in `band` doubles
inline int band_rows(int U, int r0, int band) {
  int64_t room = band;
  int R = 0;
  while (r0 + R < U && room >= U - r0 - R) room -= U - r0 - R++;
  return R;
}
constexpr int kFullRows = 1 << 30;  // item: full rows (with R in z), not rows of the triangle

// position of (lo, hi), lo <= hi, in the row-packed upper triangle of a
// U x U block: tri_base(lo, U) + hi
__host__ __device__ inline int tri_base(int lo, int U) { return lo * (2 * U - lo + 1) / 2 - lo; }

inline unsigned nblocks(int64_t n, int b = 256) { return (unsigned)((n + b - 1) / b); }

// Pair id P = i * G + g.  Key = tube cell of x_g in the plane (2-D: on the
// line) orthogonal to e_i; x_g summed in the walk's order ((0 + b0 v0) + b1 v1) + ...
struct TubeCells {
  double lo[3], inv_c[3];  // per axis: lower end, 1 / cell edge
  int n[3];                // per axis: cells
  uint32_t per_axis;       // cells of the plane with most of them
};
__global__ void k_pair_keys(TubeGeom q, int nq, int64_t G, TubeCells cells, uint32_t *__restrict__ key,
                            int32_t *__restrict__ val) {
  const int64_t P = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (P >= q.dim * G) return;
  const int i = (int)(P / G);
  const int64_t g = P - (int64_t)i * G;
  const int64_t t = g / nq;
  const int k = (int)(g - t * nq), nv = q.dim + 1;
  double x[3] = {0.0, 0.0, 0.0};
  for (int m = 0; m < nv; m++) {
    const double b = q.rule[nv * k + m];
    const double *v = q.xyz + q.dim * (int64_t)q.elem[nv * t + m];
    x[0] = x[0] + b * v[0];
    x[1] = x[1] + b * v[1];
    if (q.dim == 3) x[2] = x[2] + b * v[2];
  }
  uint32_t id = 0;
  for (int d = 1; d < q.dim; d++) {
    const int ax = (i + d) % q.dim, n = cells.n[ax];
    const int c = (int)floor(((ax == 0 ? x[0] : (ax == 1 ? x[1] : x[2])) - cells.lo[ax]) * cells.inv_c[ax]);
    id = id * (uint32_t)n + (uint32_t)(c < 0 ? 0 : (c >= n ? n - 1 : c));
  }
  key[P] = (uint32_t)i * cells.per_axis + id;
  val[P] = (int32_t)P;
}

__global__ void k_heads(const uint32_t *__restrict__ key, int64_t n, int32_t *__restrict__ head) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n) head[k] = (k == 0 || key[k] != key[k - 1]) ? 1 : 0;
}

// tube_off[T] = first sorted position of tube T; tube_off[n_tubes] = n
__global__ void k_tube_off(const int32_t *__restrict__ head, const int32_t *__restrict__ tid, int64_t n,
                           int64_t *__restrict__ tube_off) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n && head[k]) tube_off[tid[k]] = k;
  if (k == n - 1) tube_off[tid[k] + head[k]] = n;
}

// per sorted pair: {l first entry, r first entry, |l|, |r| | axis << 30} and w_g
__global__ void k_pair_meta(const int32_t *__restrict__ pair_sorted, int64_t n, int64_t G, int nq,
                            const int64_t *__restrict__ off, const double *__restrict__ qw,
                            const double *__restrict__ vol, int4 *__restrict__ pm, double *__restrict__ pw) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const int64_t P = pair_sorted[k];
  const int i = (int)(P / G);
  const int64_t g = P - (int64_t)i * G;
  const int64_t hl = (int64_t)(2 * i) * G + g, hr = hl + G;
  int4 m;
  m.x = (int)off[hl];
  m.y = (int)off[hr];
  m.z = (int)(off[hl + 1] - off[hl]);
  m.w = (int)(off[hr + 1] - off[hr]) | (i << 30);
  pm[k] = m;
  const int64_t t = g / nq;
  pw[k] = qw[g - t * nq] * vol[t];
}

__device__ __forceinline__ unsigned hash_slot(int32_t d) { return ((uint32_t)d * 2654435761u) >> (32 - 13); }

// insert every node of the tube's entries into the LDS hash; returns through
// `cnt` the number of distinct nodes, or more than kMaxTube as soon as there are:
// the table stays about half full (a full one would be probed all round by every
// further node: minutes on a strip of 4 200 x 3 cells, whose chords have 8 400)
__device__ void tube_insert(int32_t *hk, int *cnt, const int4 *__restrict__ pm, int64_t k0, int64_t k1,
                            const int32_t *__restrict__ ent_dof) {
  for (int j = threadIdx.x; j < kHash; j += blockDim.x) hk[j] = -1;
  if (threadIdx.x == 0) *cnt = 0;
  __syncthreads();
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  for (int64_t k = k0 + wave; k < k1; k += nw) {
    const int4 m = pm[k];
    const int nl = m.z, nr = m.w & 0x3fffffff;
    for (int e = lane; e < nl + nr; e += 64) {
      if (*(volatile int *)cnt > kMaxTube) {
        k = k1;
        break;
      }
      const int32_t d = ent_dof[e < nl ? m.x + e : m.y + (e - nl)];
      unsigned h = hash_slot(d);
      for (int probe = 0; probe < kHash; probe++) {
        const int32_t old = atomicCAS(&hk[h], -1, d);
        if (old == -1) {
          atomicAdd(cnt, 1);
          break;
        }
        if (old == d) break;
        h = (h + 1) & (kHash - 1);
      }
    }
  }
  __syncthreads();
}

// threads of a tube's count and fill: few tubes of many nodes leave the chip to
// one workgroup per tube
constexpr int kPlanThreads = 1024;

__global__ void __launch_bounds__(kPlanThreads) k_tube_count(const int64_t *__restrict__ tube_off, const int4 *__restrict__ pm,
                                                    const int32_t *__restrict__ ent_dof, int64_t *__restrict__ u_cnt,
                                                    int32_t *flag) {
  __shared__ int32_t hk[kHash];
  __shared__ int cnt;
  const int64_t T = blockIdx.x;
  tube_insert(hk, &cnt, pm, tube_off[T], tube_off[T + 1], ent_dof);
  if (threadIdx.x == 0) {
    u_cnt[T] = cnt;
    if (cnt > kMaxTube) set_flag(flag, FPDE_EUNSUPPORTED);
  }
}

// U_T sorted, the slot of every entry, and per-row counts of (tube, slot) places
__global__ void __launch_bounds__(kPlanThreads) k_tube_fill(const int64_t *__restrict__ tube_off, const int4 *__restrict__ pm,
                                                   const int32_t *__restrict__ ent_dof,
                                                   const int64_t *__restrict__ u_off, int32_t *__restrict__ tube_u,
                                                   int32_t *__restrict__ ent_slot, int64_t *__restrict__ row_cnt) {
  __shared__ int32_t hk[kHash];
  __shared__ int32_t su[kMaxTube];
  __shared__ int cnt, cnt2;
  const int64_t T = blockIdx.x;
  const int64_t k0 = tube_off[T], k1 = tube_off[T + 1];
  tube_insert(hk, &cnt, pm, k0, k1, ent_dof);
  const int U = cnt;
  int P2 = 1;
  while (P2 < U) P2 <<= 1;
  if (threadIdx.x == 0) cnt2 = 0;
  __syncthreads();
  for (int j = threadIdx.x; j < kHash; j += blockDim.x)
    if (hk[j] >= 0) su[atomicAdd(&cnt2, 1)] = hk[j];
  __syncthreads();
  for (int j = U + threadIdx.x; j < P2; j += blockDim.x) su[j] = 0x7fffffff;
  __syncthreads();
  // bitonic sort of su[0, P2)
  for (int size = 2; size <= P2; size <<= 1)
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      for (int j = threadIdx.x; j < P2; j += blockDim.x) {
        const int o = j ^ stride;
        if (o > j) {
          const bool up = (j & size) == 0;
          const int32_t x = su[j], y = su[o];
          if ((x > y) == up) {
            su[j] = y;
            su[o] = x;
          }
        }
      }
      __syncthreads();
    }
  const int64_t ub = u_off[T];
  for (int j = threadIdx.x; j < U; j += blockDim.x) {
    tube_u[ub + j] = su[j];
    atomicAdd((unsigned long long *)&row_cnt[su[j]], 1ull);
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  for (int64_t k = k0 + wave; k < k1; k += nw) {
    const int4 m = pm[k];
    const int nl = m.z, nr = m.w & 0x3fffffff;
    for (int e = lane; e < nl + nr; e += 64) {
      const int64_t ei = e < nl ? m.x + e : m.y + (e - nl);
      const int32_t d = ent_dof[ei];
      int lo = 0, hi = U - 1;
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (su[mid] < d) lo = mid + 1;
        else hi = mid;
      }
      ent_slot[ei] = lo;
    }
  }
}

__global__ void k_row_places(const int64_t *__restrict__ u_off, int64_t n_tubes, const int32_t *__restrict__ tube_u,
                             int64_t *__restrict__ cursor, int2 *__restrict__ row_ts) {
  const int64_t T = blockIdx.x;
  if (T >= n_tubes) return;
  const int64_t u0 = u_off[T], U = u_off[T + 1] - u0;
  for (int64_t s = threadIdx.x; s < U; s += blockDim.x) {
    const int32_t d = tube_u[u0 + s];
    const unsigned long long pos = atomicAdd((unsigned long long *)&cursor[d], 1ull);
    row_ts[pos] = make_int2((int)T, (int)s);
  }
}

__global__ void k_block_sizes(const int64_t *__restrict__ u_off, int64_t n_tubes, int64_t *__restrict__ usq) {
  const int64_t T = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (T >= n_tubes) return;
  const int64_t U = u_off[T + 1] - u_off[T];
  usq[T] = U * U;
}

struct AccumArgs {
  const int64_t *tube_off;
  const int4 *pm;
  const double *pw;
  const int4 *items;
  const int32_t *ent_slot;
  const double *ent_val;
  const int64_t *blk_off;
  double *blk;
  double KC0, KC1, KC2;
  // general form (k_tube_form): test-order values, constant coefficients, and
  // coefficients per pair (id i G + g, those of cr after ncoef of cl) or null
  const double *val_b;
  const int32_t *pair;
  const double *coef;
  int64_t ncoef;
  double cl0, cl1, cl2, cr0, cr1, cr2;
};

__device__ __forceinline__ int pair_nl(const int4 &m) { return m.z; }
__device__ __forceinline__ int pair_nr(const int4 &m) { return m.w & 0x3fffffff; }

// ---- Outer products of half-ray vectors into an LDS band ----
//
// A wavefront takes one pair at a time, in steps of up to 64 entries of one
// side (rows) times 64 of the other (columns), as tiles of 16 rows x 4
// columns: lane l holds row entry 16 i + (l & 15) of the step in four copies,
// and column entry 4 (l & 15) + (l >> 4), so that each group of 16 lanes finds
// its column of tile column t in its own lane t (a row broadcast, no LDS and
// no scalar registers).  A tile is one product, three integer operations for
// the address and one LDS update of up to 64 distinct lanes.  (One row entry
// per lane, with the columns broadcast one at a time, filled 18 of 64 lanes at
// 20 instructions an update.)  The entries of the next two steps are in flight
// while a step is multiplied, and the next pair's metadata beyond them.
//   kSquare: the whole block, row stride Up, each product once at (min, max);
//   kTri:    the same as a row-packed upper triangle;
//   kTriBand: rows [r0, r0 + R) of that triangle (products with their smaller
//            slot elsewhere are left out);
//   kFull:   block rows [r0, r0 + R), row stride Up, both products of a pair
//            (rows l, columns r, then rows r, columns l).
// Measured rates: an LDS update of 64 lanes issues every 3.9 ns per CU, of 18
// lanes every 3.0 ns; same-address lanes of one update are served one by one.
enum BandLayout { kSquare = 0, kTri = 1, kTriBand = 2, kFull = 3 };

constexpr int kStep = 64;  // entries of each side in one step

struct PairStep {
  int rs[4], cs;      // slots, in bytes of a row of doubles
  double rv[4], cv;   // values
  int nr, nc;         // entries of each side
  double w;           // weight of the products
};

// entry k of a side [e0, e0 + n), clamped into it (entry 0 for an empty side,
// whose offset may equal the entry count); lanes past the end are masked
__device__ __forceinline__ int side_entry(int e0, int n, int k) { return n > 0 ? e0 + (k < n ? k : n - 1) : 0; }

// The steps of one wavefront: pairs k, k + nw, ..., and of each its roles, row
// blocks and column blocks.  Everything here is the wavefront's (scalar).
template <int ROLES>
struct StepCursor {
  const int4 *__restrict__ pm;
  const double *__restrict__ pw;
  // coefficients per pair (general form), by pair id i G + g: of role 1 at
  // coef[id], of role 0 at coef[ncoef + id]; else null
  const int32_t *__restrict__ pair;
  const double *__restrict__ coef;
  int64_t ncoef;
  int64_t k, k1;
  int nw;
  int4 m, mn;
  double w[ROLES], wn[ROLES];
  int role, rb, cb;
  __device__ __forceinline__ void fetch(int64_t kk, int4 &mm, double (&ww)[ROLES]) {
    kk = kk < k1 ? kk : k1 - 1;
    mm = pm[kk];
    ww[0] = pw[kk];
    if constexpr (ROLES == 2) {
      ww[1] = ww[0];
      if (coef) {
        const int64_t id = pair[kk];
        ww[0] *= coef[ncoef + id];
        ww[1] *= coef[id];
      }
    }
  }
  __device__ __forceinline__ double weight() const { return ROLES == 2 && role ? w[ROLES - 1] : w[0]; }
  __device__ __forceinline__ void start(int64_t k0) {
    k = k0;
    role = rb = cb = 0;
    if (k >= k1) return;
    fetch(k, m, w);
    fetch(k + nw, mn, wn);
  }
  __device__ __forceinline__ int nl() const { return pair_nl(m); }
  __device__ __forceinline__ int nr() const { return pair_nr(m); }
  __device__ __forceinline__ void next() {
    const int nrow = role ? nr() : nl(), ncol = role ? nl() : nr();
    cb += kStep;
    if (cb < ncol) return;
    cb = 0;
    rb += kStep;
    if (rb < nrow) return;
    rb = 0;
    if (++role < ROLES) return;
    role = 0;
    k += nw;
    m = mn;
#pragma unroll
    for (int q = 0; q < ROLES; q++) w[q] = wn[q];
    if (k < k1) fetch(k + nw, mn, wn);
  }
};

// entries of the cursor's step: rows from vrow, columns from vcol
template <int ROLES>
__device__ __forceinline__ void load_step(const StepCursor<ROLES> &c, const int32_t *__restrict__ slot,
                                          const double *__restrict__ vrow, const double *__restrict__ vcol,
                                          double w, PairStep &p) {
  const int lane = threadIdx.x & 63, lr = lane & 15, lc = lane >> 4;
  const int nl = c.nl(), nr = c.nr();
  const int erow = c.role ? c.m.y : c.m.x, ecol = c.role ? c.m.x : c.m.y;
  const int nrow = c.role ? nr : nl, ncol = c.role ? nl : nr;
  p.nr = nrow - c.rb < kStep ? nrow - c.rb : kStep;
  p.nc = ncol - c.cb < kStep ? ncol - c.cb : kStep;
  p.w = w;
#pragma unroll
  for (int i = 0; i < 4; i++) {
    if (i > 0 && 16 * i >= p.nr) break;
    const int er = side_entry(erow, nrow, c.rb + 16 * i + lr);
    p.rs[i] = slot[er] * 8;
    p.rv[i] = vrow[er];
  }
  const int ec = side_entry(ecol, ncol, c.cb + 4 * lr + lc);
  p.cs = slot[ec] * 8;
  p.cv = vcol[ec];
}

// lane t of each group of 16 lanes, in all of the group
template <int t>
__device__ __forceinline__ int group_lane(int v) {
  return __builtin_amdgcn_update_dpp(0, v, 0x150 + t, 0xf, 0xf, true);
}
template <int t>
__device__ __forceinline__ double group_lane(double v) {
  return __hiloint2double(group_lane<t>(__double2hiint(v)), group_lane<t>(__double2loint(v)));
}

struct Band {
  char *acc;
  int U, Up, r0, R, off;  // off: bytes of the triangle before row r0
};

// tile column t of a step with NCH chunks of 16 rows, then the next one
template <int LAYOUT, int NCH, int t>
__device__ __forceinline__ void step_columns(const Band &b, const PairStep &p, double cvw) {
  if (4 * t >= p.nc) return;
  const int lane = threadIdx.x & 63;
  const int y = group_lane<t>(p.cs);
  const double cv = group_lane<t>(cvw);
  const bool cok = 4 * t + (lane >> 4) < p.nc;
#pragma unroll
  for (int i = 0; i < NCH; i++) {
    const int x = p.rs[i];
    bool ok = cok && 16 * i + (lane & 15) < p.nr;
    int at;
    if (LAYOUT == kFull) {
      ok = ok && (unsigned)(x - 8 * b.r0) < (unsigned)(8 * b.R);
      at = (x - 8 * b.r0) * b.Up + y;
    } else {
      const int lo = x < y ? x : y, hi = x < y ? y : x;
      if (LAYOUT == kSquare) {
        at = lo * b.Up + hi;
      } else {
        if (LAYOUT == kTriBand) ok = ok && (unsigned)(lo - 8 * b.r0) < (unsigned)(8 * b.R);
        at = (lo >> 3) * (8 * b.U - 4 - (lo >> 1)) + hi;  // 8 (tri_base(lo / 8, U) + hi / 8)
        if (LAYOUT == kTriBand) at -= b.off;
      }
    }
    if (ok) atomicAdd((double *)(b.acc + at), p.rv[i] * cv);
  }
  if constexpr (t < 15) step_columns<LAYOUT, NCH, t + 1>(b, p, cvw);
}

template <int LAYOUT>
__device__ __forceinline__ void step_products(const Band &b, const PairStep &p) {
  if (p.nr <= 0) return;
  const double cvw = p.cv * p.w;
  if (p.nr <= 16) step_columns<LAYOUT, 1, 0>(b, p, cvw);
  else if (p.nr <= 32) step_columns<LAYOUT, 2, 0>(b, p, cvw);
  else if (p.nr <= 48) step_columns<LAYOUT, 3, 0>(b, p, cvw);
  else step_columns<LAYOUT, 4, 0>(b, p, cvw);
}

// Every pair of [k0, k1) into the band; kc0, kc1: the tube's coefficient in
// role 0 and 1 (its pairs share one axis).
template <int LAYOUT>
__device__ __forceinline__ void band_products(double *acc, int U, int Up, int r0, int R, const AccumArgs &a,
                                              const double *__restrict__ vrow, const double *__restrict__ vcol,
                                              double kc0, double kc1, int64_t k0, int64_t k1) {
  constexpr int ROLES = LAYOUT == kFull ? 2 : 1;
  // wave-uniform (readfirstlane), so the cursor and its loads are scalar
  StepCursor<ROLES> c;
  c.pm = a.pm;
  c.pw = a.pw;
  c.pair = a.pair;
  c.coef = a.coef;
  c.ncoef = a.ncoef;
  c.k1 = k1;
  c.nw = blockDim.x >> 6;
  c.start(k0 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6));
  const Band b = {(char *)acc, U, Up, r0, R, 8 * (tri_base(r0, U) + r0)};
  auto load = [&](PairStep &p) {
    p.nr = 0;
    if (c.k >= k1) return false;
    load_step(c, a.ent_slot, vrow, vcol, c.weight() * (c.role ? kc1 : kc0), p);
    c.next();
    return true;
  };
  PairStep s0, s1, s2;
  if (!load(s0)) return;
  load(s1);
  for (;;) {
    const bool more = load(s2);
    step_products<LAYOUT>(b, s0);
    s0 = s1;
    s1 = s2;
    if (!more && s0.nr <= 0 && s1.nr <= 0) break;
  }
}

// lane q + rank of the set lanes gets the rank-th set lane's v (all 64 lanes take
// part: the others follow behind, so that to[] is a permutation of the wavefront)
__device__ __forceinline__ int push_lane(int to, int v) { return __builtin_amdgcn_ds_permute(4 * to, v); }
__device__ __forceinline__ double push_lane(int to, double v) {
  return __hiloint2double(push_lane(to, __double2hiint(v)), push_lane(to, __double2loint(v)));
}

// Every pair of [k0, k1) into block rows [r0, r0 + R), both products: the entries
// of a half-ray that stand in these rows are collected first, up to 64 in the
// wavefront's registers, then multiplied by every entry of the other side.  For
// bands of few rows: bound by the products (LDS updates); with every product tried
// against the band, as band_products does, 3 x 3 x 400 cells took 200 times as long.
__device__ __forceinline__ void row_products(double *acc, int U, int Up, int r0, int R, const AccumArgs &a,
                                             const double *__restrict__ vrow, const double *__restrict__ vcol,
                                             double kc0, double kc1, int64_t k0, int64_t k1) {
  const int lane = threadIdx.x & 63, nw = blockDim.x >> 6;
  const int32_t *__restrict__ slot = a.ent_slot;
  const Band b = {(char *)acc, U, Up, r0, R, 0};
  for (int64_t k = k0 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); k < k1; k += nw) {
    const int4 m = a.pm[k];
    const int nl = pair_nl(m), nr = pair_nr(m);
    double w0 = a.pw[k] * kc0, w1 = a.pw[k] * kc1;
    if (a.coef) {
      const int64_t id = a.pair[k];
      w0 *= a.coef[a.ncoef + id];
      w1 *= a.coef[id];
    }
#pragma unroll 1
    for (int role = 0; role < 2; role++) {
      const int erow = role ? m.y : m.x, ecol = role ? m.x : m.y;
      const int nrow = role ? nr : nl, ncol = role ? nl : nr;
      if (ncol == 0) continue;
      const double w = role ? w1 : w0;
      int qn = 0, qs = 0;  // the rows collected: lanes 0 .. qn - 1
      double qv = 0.0;
      auto flush = [&]() {
        PairStep p;
        p.nr = qn;
#pragma unroll
        for (int i = 0; i < 4; i++) {
          p.rs[i] = __shfl(qs, 16 * i + (lane & 15), 64) * 8;
          p.rv[i] = __shfl(qv, 16 * i + (lane & 15), 64);
        }
        const int at = 4 * (lane & 15) + (lane >> 4);
        int ec = side_entry(ecol, ncol, at);
        int cs = slot[ec];
        double cv = vcol[ec];
        for (int cb = 0; cb < ncol; cb += kStep) {
          p.nc = ncol - cb < kStep ? ncol - cb : kStep;
          p.cs = cs * 8;
          p.cv = cv;
          p.w = w;
          ec = side_entry(ecol, ncol, cb + kStep + at);
          cs = slot[ec];
          cv = vcol[ec];
          step_products<kFull>(b, p);
        }
      };
      int sn = slot[side_entry(erow, nrow, lane)];
      for (int j0 = 0; j0 < nrow; j0 += 64) {
        const int s = sn;
        sn = slot[side_entry(erow, nrow, j0 + 64 + lane)];
        const bool in = j0 + lane < nrow && (unsigned)(s - r0) < (unsigned)R;
        const uint64_t bal = __ballot(in);
        if (bal == 0) continue;
        const double v = vrow[side_entry(erow, nrow, j0 + lane)];
        const int cnt = __popcll(bal);
        const int rank = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
        const int to = (in ? qn + rank : qn + cnt + lane - rank) & 63;
        const int ms = push_lane(to, s);
        const double mv = push_lane(to, v);
        if (lane >= qn) {
          qs = ms;
          qv = mv;
        }
        qn += cnt;
        if (qn >= 64) {
          const int over = qn - 64;
          qn = 64;
          flush();
          qn = over;  // the rest came round to the first lanes
          qs = ms;
          qv = mv;
        }
      }
      if (qn > 0) flush();
    }
  }
}

__global__ void __launch_bounds__(kAccumThreads) k_tube_accum(AccumArgs a) {
  extern __shared__ double acc[];
  const int4 it = a.items[blockIdx.x];
  const int64_t T = it.x;
  const int r0 = it.y, R = it.z & ~kFullRows, U = it.w, Up = band_stride(U);
  // B = S + S^T with S = sum_p w_p l_p r_p^T: each product of S once, at
  // (min, max), half the LDS updates of the two products, in the full square
  // when it fits (no bank conflicts and the cheaper address), else in the
  // packed triangle or half of it; larger blocks by full rows
  const bool full = it.z & kFullRows, square = R == U && U * Up <= kBand;
  const int tri0 = tri_base(r0, U) + r0;
  const int nacc = square || full ? R * Up : tri_base(r0 + R, U) + r0 + R - tri0;
  for (int j = threadIdx.x; j < nacc; j += blockDim.x) acc[j] = 0.0;
  __syncthreads();
  const int64_t k0 = a.tube_off[T], k1 = a.tube_off[T + 1];
  const int axis = (int)((unsigned)a.pm[k0].w >> 30);  // a tube has at least one pair
  const double kc = axis == 0 ? a.KC0 : (axis == 1 ? a.KC1 : a.KC2);
  if (full && 3 * R >= U) band_products<kFull>(acc, U, Up, r0, R, a, a.ent_val, a.ent_val, kc, kc, k0, k1);
  else if (full) row_products(acc, U, Up, r0, R, a, a.ent_val, a.ent_val, kc, kc, k0, k1);
  else if (square) band_products<kSquare>(acc, U, Up, r0, R, a, a.ent_val, a.ent_val, kc, kc, k0, k1);
  else if (R == U) band_products<kTri>(acc, U, Up, r0, R, a, a.ent_val, a.ent_val, kc, kc, k0, k1);
  else band_products<kTriBand>(acc, U, Up, r0, R, a, a.ent_val, a.ent_val, kc, kc, k0, k1);
  __syncthreads();
  const int lane = threadIdx.x & 63;
  double *blk = a.blk + a.blk_off[T];
  if (full) {
    for (int i = threadIdx.x >> 6; i < R; i += blockDim.x >> 6)
      for (int t = lane; t < U; t += 64) blk[(int64_t)(r0 + i) * U + t] = acc[i * Up + t];
    return;
  }
  // every entry whose smaller index lies in the band, one wavefront per row
  for (int i = r0 + (threadIdx.x >> 6); i < U; i += blockDim.x >> 6) {
    double *out = blk + (int64_t)i * U;
    const int t1 = i < r0 + R ? U : r0 + R;
    for (int t = r0 + lane; t < t1; t += 64) {
      const int lo = i < t ? i : t, hi = i < t ? t : i;
      const double v = acc[(square ? lo * Up : tri_base(lo, U) - tri0) + hi];
      out[t] = i == t ? v + v : v;
    }
  }
}

// General form (Sec. 1, the test operator on the side opposite to the trial
// one), with constant coefficients or one per Gauss point and axis: per pair, with l / r the left / right
// half-rays, the trial values at orders alpha (a.ent_val) and the test
// values at orders beta (a.val_b),
//   B[k][l] += w cl_i r_beta[k] l_alpha[l] + w cr_i l_beta[k] r_alpha[l]
// (rows: test node, columns: trial node).  Not symmetric, so both products
// of every pair go into full rows.
__global__ void __launch_bounds__(kAccumThreads) k_tube_form(AccumArgs a) {
  extern __shared__ double acc[];
  const int4 it = a.items[blockIdx.x];
  const int64_t T = it.x;
  const int r0 = it.y, R = it.z, U = it.w, Up = band_stride(U);
  const int64_t k0 = a.tube_off[T], k1 = a.tube_off[T + 1];
  // role 0: rows l (beta), columns r (alpha, cr); role 1: rows r, columns l (cl)
  const int axis = (int)((unsigned)a.pm[k0].w >> 30);
  const double kc0 = a.coef ? 1.0 : (axis == 0 ? a.cr0 : (axis == 1 ? a.cr1 : a.cr2));
  const double kc1 = a.coef ? 1.0 : (axis == 0 ? a.cl0 : (axis == 1 ? a.cl1 : a.cl2));
  for (int j = threadIdx.x; j < R * Up; j += blockDim.x) acc[j] = 0.0;
  __syncthreads();
  if (3 * R >= U) band_products<kFull>(acc, U, Up, r0, R, a, a.val_b, a.ent_val, kc0, kc1, k0, k1);
  else row_products(acc, U, Up, r0, R, a, a.val_b, a.ent_val, kc0, kc1, k0, k1);
  __syncthreads();
  double *out = a.blk + a.blk_off[T] + (int64_t)r0 * U;
  for (int i = threadIdx.x >> 6; i < R; i += blockDim.x >> 6)
    for (int t = threadIdx.x & 63; t < U; t += 64) out[(int64_t)i * U + t] = acc[i * Up + t];
}

struct GatherArgs {
  const int64_t *row_off;
  const int2 *row_ts;
  const int64_t *u_off;
  const int32_t *tube_u;
  const int64_t *blk_off;
  const double *blk;
  // per tube, the first position in U_T of every column chunk: cstart[T
  // (nch + 1) + c] = #{nodes of U_T below c chunk} (U_T is increasing)
  const int32_t *cstart;
  int64_t ndof, lda;
  int chunk, nch;
};

// cstart for every (tube, chunk boundary): a binary search in U_T
__global__ void k_chunk_starts(const int64_t *__restrict__ u_off, const int32_t *__restrict__ tube_u, int64_t n_tubes,
                               int chunk, int nch, int32_t *__restrict__ cstart) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_tubes * (nch + 1)) return;
  const int64_t T = i / (nch + 1);
  const int64_t lim = (int64_t)(i % (nch + 1)) * chunk;
  int64_t lo = u_off[T], hi = u_off[T + 1];
  const int64_t first = lo;
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if (tube_u[mid] < lim) lo = mid + 1;
    else hi = mid;
  }
  cstart[i] = (int32_t)(lo - first);
}

__device__ __forceinline__ int64_t lane64(int64_t v, int l) {
  const int lo = __builtin_amdgcn_readlane((int)(uint32_t)v, l);
  const int hi = __builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)v >> 32), l);
  return (int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}

// Row `row`, column chunk ci ([c0, c0 + cw)) of K into the LDS chunk racc:
// the sum over the (tube, slot) places of the node of that slot's row of
// the tube block, scattered through U_T (one wavefront per place).  Only
// the part of the block row whose nodes fall in the chunk is read (U_T is
// increasing, so it is the range [cstart(T, ci), cstart(T, ci + 1))).  The
// places' metadata (tube, slot, node-set offset, block offset, range) is
// loaded 64 places at a time, one per lane, and broadcast from there.
// Ends with the chunk complete and visible to the whole workgroup.
__device__ __forceinline__ void gather_row_chunk(const GatherArgs &a, int64_t row, int ci, int64_t c0, int64_t cw,
                                                 double *racc) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nwave = blockDim.x >> 6;
  const int64_t p0 = a.row_off[row], np = a.row_off[row + 1] - p0;
  for (int64_t j = threadIdx.x; j < cw; j += blockDim.x) racc[j] = 0.0;
  __syncthreads();
  for (int64_t pb = 0; pb < np; pb += 64) {
    int64_t u0 = 0, brow0 = 0;
    int t0 = 0, t1 = 0;
    if (pb + lane < np) {
      const int2 ts = a.row_ts[p0 + pb + lane];
      u0 = a.u_off[ts.x];
      const int64_t U = a.u_off[ts.x + 1] - u0;
      brow0 = a.blk_off[ts.x] + (int64_t)ts.y * U;
      const int32_t *cs = a.cstart + (int64_t)ts.x * (a.nch + 1) + ci;
      t0 = cs[0];
      t1 = cs[1];
    }
    const int cnt = (int)((np - pb) < 64 ? (np - pb) : 64);
    for (int k = wave; k < cnt; k += nwave) {
      const int64_t uk = lane64(u0, k);
      const double *brow = a.blk + lane64(brow0, k);
      const int tk1 = __builtin_amdgcn_readlane(t1, k);
      for (int t = __builtin_amdgcn_readlane(t0, k) + lane; t < tk1; t += 64)
        atomicAdd(&racc[(int64_t)a.tube_u[uk + t] - c0], brow[t]);
    }
  }
  __syncthreads();
}

// row of the dealt slot b: rows dealt XCD by XCD in contiguous ranges
// (workgroups go round-robin to the 8 XCDs)
__device__ __forceinline__ int64_t dealt_row(int64_t b, int64_t ndof) {
  const int64_t per_xcd = (ndof + 7) / 8;
  return (b % 8) * per_xcd + b / 8;
}

// A[p, :] = row p of K, written densely, once.
template <class TO>
__global__ void __launch_bounds__(256) k_tube_gather(GatherArgs a, TO *__restrict__ A) {
  extern __shared__ double racc[];
  const int64_t slots = 8 * ((a.ndof + 7) / 8);
  for (int64_t b = blockIdx.x; b < slots; b += gridDim.x) {
    const int64_t row = dealt_row(b, a.ndof);
    if (row >= a.ndof) continue;
    for (int ci = 0; ci < a.nch; ci++) {
      const int64_t c0 = (int64_t)ci * a.chunk;
      const int64_t cw = (a.ndof - c0) < a.chunk ? (a.ndof - c0) : a.chunk;
      gather_row_chunk(a, row, ci, c0, cw, racc);
      TO *out = A + row * a.lda + c0;
      for (int64_t j = threadIdx.x; j < cw; j += blockDim.x) out[j] = (TO)racc[j];
      __syncthreads();
    }
  }
}

// The same rows, kept only at the columns of a CSR pattern (sorted columns
// per row): val[q] = K[row, col[q]] for q in [row_ptr[row], row_ptr[row+1]).
__global__ void __launch_bounds__(256) k_tube_gather_csr(GatherArgs a, const int64_t *__restrict__ row_ptr,
                                                         const int32_t *__restrict__ col,
                                                         double *__restrict__ val) {
  extern __shared__ double racc[];
  const int64_t slots = 8 * ((a.ndof + 7) / 8);
  for (int64_t b = blockIdx.x; b < slots; b += gridDim.x) {
    const int64_t row = dealt_row(b, a.ndof);
    if (row >= a.ndof) continue;
    const int64_t q0 = row_ptr[row], q1 = row_ptr[row + 1];
    for (int ci = 0; ci < a.nch; ci++) {
      const int64_t c0 = (int64_t)ci * a.chunk;
      const int64_t cw = (a.ndof - c0) < a.chunk ? (a.ndof - c0) : a.chunk;
      gather_row_chunk(a, row, ci, c0, cw, racc);
      for (int64_t q = q0 + threadIdx.x; q < q1; q += blockDim.x) {
        const int64_t d = (int64_t)col[q] - c0;
        if ((uint64_t)d < (uint64_t)cw) val[q] = racc[d];
      }
      __syncthreads();
    }
  }
}

// ---- Tube blocks on the matrix cores in split FP16 (mixed precision) ----
//
// The block of a tube is one product B = X Y^T with an inner dimension of
// two columns per pair p: X_{:,2p} = W_p l_p, X_{:,2p+1} = W_p r_p,
// Y_{:,2p} = r_p, Y_{:,2p+1} = l_p (W_p = w_g K_i c_alpha), so that
// (X Y^T)_jk = sum_p W_p (l_j r_k + r_j l_k): the L W R^T contraction of the
// element quadrature, symmetric.  A node appears several times in one
// half-ray (once per element the ray crosses around it); those entries are
// summed first (in FP64, per assembly), so that a pair's side has one
// merged entry per node and every inner column of X and Y receives each of
// its rows at most once.  One workgroup (eight wavefronts, 64 x 32 each)
// computes a 128 x 128 region (I, J), I <= J, of B and writes it and its
// mirror into the tube's block.  The pairs go through LDS sixteen at a
// time (32 inner columns, one depth of v_mfma_f32_16x16x32_f16): the merged
// entries, scaled by the tube's powers of two (largest magnitude of X and
// of Y in [2^13, 2^14)), are split into FP16 hi + lo and stored straight
// into the operand panels, and the region accumulates hi hi + hi lo + lo hi
// in FP32 (22 significant bits per operand; the dropped lo lo term is
// below 2^-22 of each product).
constexpr int kRegion = 128;
constexpr int kChunkPairs = 16;
constexpr int kTubeThreads = 512;  // eight wavefronts per region, 64 x 32 of it each
constexpr int kMergeSlots = 4096;  // largest tube (|U_T|) of the matrix-core path
constexpr int kMergeMax = 512;     // most merged entries of one pair on that path

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float f32x4v __attribute__((ext_vector_type(4)));

// 16-byte group q of row `row` (64-byte rows): q ^ h(row) with
// h = (r1 ^ r2) | (r1 ^ r3) << 1 over the row's bits, so the lanes of one
// operand read (16 consecutive rows, one q) hit distinct 16-byte slots
// whether the LDS serves them 8 at a time in a 128-byte window or 16 at a
// time in a 256-byte window
__device__ __forceinline__ int tswz(int row, int q) {
  return q ^ ((((row >> 1) ^ (row >> 2)) & 1) | ((((row >> 1) ^ (row >> 3)) & 1) << 1));
}

// [buffer][hi, lo][row][16-byte group]: declared as 16-byte groups so that
// the operand reads are single ds_read_b128
struct TubeMfmaSmem {
  half8 hx[2][2][kRegion][2 * kChunkPairs / 8];
  half8 hy[2][2][kRegion][2 * kChunkPairs / 8];
};

// Merge structure of every sorted pair (plan time), one wavefront per pair:
// the merged entries of a side are its distinct tube slots in order of first
// occurrence (l's first, then r's).  COUNT: cnt[k] = the pair's merged
// entries.  FILL: for every entry its merged index within the pair (midx),
// and per merged entry slot | (inner column << 16), the column being
// 2 (pair mod 16) + side; the pair's tube into pk_tube.  Slots must be below
// kMergeSlots; COUNT also takes into *maxc (zero on entry) the largest count
// above kMergeMax.
template <bool FILL>
__global__ void __launch_bounds__(64) k_merge_pairs(const int64_t *__restrict__ tube_off, int64_t n_tubes,
                                                    const int4 *__restrict__ pm, int64_t n_pairs,
                                                    const int32_t *__restrict__ ent_slot, int64_t *__restrict__ cnt,
                                                    const int64_t *__restrict__ mk_pair, uint16_t *__restrict__ midx,
                                                    uint32_t *__restrict__ mk_meta, int32_t *__restrict__ pk_tube,
                                                    int *__restrict__ maxc) {
  __shared__ int tbl[kMergeSlots];
  const int lane = threadIdx.x;
  const int64_t k = blockIdx.x;
  if (k >= n_pairs) return;  // the whole block (one wavefront)
  const int4 m = pm[k];
  uint32_t col0 = 0;
  if (FILL) {
    int64_t lo = 0, hi = n_tubes - 1;  // the pair's tube: the last T with tube_off[T] <= k
    while (lo < hi) {
      const int64_t mid = (lo + hi + 1) >> 1;
      if (tube_off[mid] <= k) lo = mid;
      else hi = mid - 1;
    }
    col0 = 2u * (uint32_t)((k - tube_off[lo]) % kChunkPairs);
    if (lane == 0) pk_tube[k] = (int32_t)lo;
  }
  int merged = 0;
  for (int side = 0; side < 2; side++) {
    const int64_t base = side ? (int64_t)m.y : (int64_t)m.x;
    const int n = side ? pair_nr(m) : pair_nl(m);
    for (int e = lane; e < n; e += 64) tbl[ent_slot[base + e]] = INT_MAX;
    __syncthreads();
    for (int e = lane; e < n; e += 64) atomicMin(&tbl[ent_slot[base + e]], e);
    __syncthreads();
    // first occurrences in order; each overwrites its slot's cell with
    // -(merged index + 1) (no other entry of that slot can be a first)
    for (int e0 = 0; e0 < n; e0 += 64) {
      const int e = e0 + lane;
      const int sl = e < n ? ent_slot[base + e] : 0;
      const bool first = e < n && tbl[sl] == e;
      const uint64_t bal = __ballot(first);
      const int r = merged + __popcll(bal & ((1ull << lane) - 1ull));
      if (first) {
        tbl[sl] = -(r + 1);
        if (FILL) {
          const int64_t q = mk_pair[k] + r;
          mk_meta[q] = (uint32_t)sl | ((col0 + (uint32_t)side) << 16);
        }
      }
      merged += __popcll(bal);
    }
    __syncthreads();
    if (FILL)
      for (int e = lane; e < n; e += 64) midx[base + e] = (uint16_t)(-tbl[ent_slot[base + e]] - 1);
    __syncthreads();
  }
  if (!FILL && lane == 0) {
    cnt[k] = merged;
    if (merged > kMergeMax) atomicMax(maxc, merged);  // only the pairs over the limit
  }
}

__global__ void k_fill_int2(int2 *__restrict__ p, int64_t n, int2 v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// Orders a wavefront's LDS accesses before and after it (no other
// wavefront shares the data).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// The merged values (every assembly): each entry's value added in FP64 into
// its merged entry (LDS) and rounded to FP32 (mk_val); and per tube the
// largest binary exponents of X (W_p |v|) and of Y (|v|) over the merged
// values: texp must hold {INT_MIN, INT_MIN} per tube on entry and receives
// atomic maxima (ilogb is monotone, so the maximum of the exponents is the
// exponent of the maximum).  Every wavefront walks pairs k = wave, wave +
// waves, ... with the next pair's metadata loaded while the current one is
// merged; its LDS row is its own, so no workgroup barrier is needed (a
// wavefront's LDS operations complete in order).
__global__ void __launch_bounds__(256) k_merge_vals(const int4 *__restrict__ pm, const double *__restrict__ pw,
                                                    const int64_t *__restrict__ mk_pair,
                                                    const int32_t *__restrict__ pk_tube,
                                                    const uint16_t *__restrict__ midx, int64_t n_pairs,
                                                    const double *__restrict__ val, double KC0, double KC1, double KC2,
                                                    float *__restrict__ mk_val, int2 *__restrict__ texp) {
  __shared__ double acc[4][kMergeMax];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t waves = (int64_t)gridDim.x * 4;
  double *a = acc[w];
  int64_t k = (int64_t)blockIdx.x * 4 + w;
  int4 m{};
  int64_t b0 = 0, b1 = 0;
  double wk = 0.0;
  int tube = 0;
  auto meta = [&](int64_t kk, int4 &mm, int64_t &c0, int64_t &c1, double &ww, int &tt) {
    if (kk < n_pairs) {
      mm = pm[kk];
      c0 = mk_pair[kk];
      c1 = mk_pair[kk + 1];
      ww = pw[kk];
      tt = pk_tube[kk];
    }
  };
  meta(k, m, b0, b1, wk, tube);
  for (; k < n_pairs; k += waves) {
    const int nm = (int)(b1 - b0);
    for (int j = lane; j < nm; j += 64) a[j] = 0.0;
    wave_lds_sync();
    // entries e < nl of l, then of r, 256 at a time: all loads of a round
    // issued before its additions; the next pair's metadata is requested
    // after the first round, so waiting for that round leaves it in flight
    const int nl = pair_nl(m), ne = nl + pair_nr(m);
    int mi[4];
    double v[4];
    auto load_round = [&](int e0) {
#pragma unroll
      for (int j = 0; j < 4; j++) {
        const int e = e0 + lane + 64 * j;
        const int64_t ei = e < nl ? (int64_t)m.x + e : (int64_t)m.y + (e - nl);
        mi[j] = e < ne ? (int)midx[ei] : -1;
        v[j] = e < ne ? val[ei] : 0.0;
      }
    };
    auto add_round = [&]() {
#pragma unroll
      for (int j = 0; j < 4; j++)
        if (mi[j] >= 0) atomicAdd(&a[mi[j]], v[j]);
    };
    load_round(0);
    int4 mn{};
    int64_t n0 = 0, n1 = 0;
    double wn = 0.0;
    int tn = 0;
    meta(k + waves, mn, n0, n1, wn, tn);
    add_round();
    for (int e0 = 256; e0 < ne; e0 += 256) {
      load_round(e0);
      add_round();
    }
    wave_lds_sync();
    float vm = 0.f;
    for (int j = lane; j < nm; j += 64) {
      const float fv = (float)a[j];
      mk_val[b0 + j] = fv;
      vm = fmaxf(vm, fabsf(fv));
    }
    wave_lds_sync();
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) vm = fmaxf(vm, __shfl_xor(vm, o, 64));
    if (lane == 0 && vm > 0.f) {
      const int axis = (int)((unsigned)m.w >> 30);
      const double mx = fabs(wk) * fabs(axis == 0 ? KC0 : (axis == 1 ? KC1 : KC2)) * (double)vm;
      int *te = (int *)&texp[tube];
      if (mx > 0.0) atomicMax(te, ilogb(mx));
      atomicMax(te + 1, ilogb((double)vm));
    }
    m = mn;
    b0 = n0;
    b1 = n1;
    wk = wn;
    tube = tn;
  }
}

// scale exponent of an operand from its largest exponent: the largest
// magnitude lands in [2^13, 2^14) (0 for an all-zero operand)
__device__ __forceinline__ int tube_scale_exp(int e) {
  if (e == INT_MIN) return 0;
  e -= 13;
  return e < -120 ? -120 : (e > 120 ? 120 : e);
}

// ---- The matrix-free product by tubes ----
//
// y = K x from the half-ray vectors: per pair the dots l.x and r.x, then
//   y += w K_i c_alpha ((r.x) l + (l.x) r).
// A tube's pairs touch only U_T, so a workgroup takes a segment of one tube's
// pairs with x on U_T and its part of y in LDS, and every entry (slot and
// value, 12 bytes) is read once, coalesced, and held in registers between its
// dot and its addition.  Groups of 16 lanes take one pair each; the groups of
// a segment start at different quarters of it, so that they seldom meet in one
// node.  Each wavefront has its own part of y (its LDS updates complete in
// order, so the sums have a fixed order); the segment's parts go to
// scratch and k_tube_sum adds them up per node.  (One pass for the dots and
// one over the node -> entry transpose, as the product went before, gathered a
// partner dot per entry: 0.37 ms against 0.11 ms for 42 077 elements.)
constexpr int kApplyHeld = 4;  // entries per lane and side held in registers
constexpr int kApplyWaves = 4;

struct ApplyArgs {
  const int4 *items;       // {tube, first pair, past the last pair, segment of the tube}
  const int4 *pm;
  const double *pw;
  const int64_t *u_off;
  const int32_t *tube_u;
  const int64_t *seg_off;  // per tube: first double of its segments' parts
  const int32_t *ent_slot;
  const double *ent_val;
  const double *x;
  double *part;
  double KC0, KC1, KC2;
  int max_u;
  CgStep cg;
};

template <int ctrl>
__device__ __forceinline__ double dpp_f64(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), ctrl, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), ctrl, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}

// sum over a group of 16 lanes, in all of them (rotations within the row)
__device__ __forceinline__ double group_sum(double v) {
  v += dpp_f64<0x128>(v);
  v += dpp_f64<0x124>(v);
  v += dpp_f64<0x122>(v);
  v += dpp_f64<0x121>(v);
  return v;
}

struct HeldSide {
  int e0, n;
  int s[kApplyHeld];
  double v[kApplyHeld];
};

__device__ __forceinline__ void held_load(HeldSide &h, int e0, int n, const int32_t *__restrict__ slot,
                                          const double *__restrict__ val) {
  const int gl = threadIdx.x & 15;
  h.e0 = e0;
  h.n = n;
#pragma unroll
  for (int j = 0; j < kApplyHeld; j++) {
    h.s[j] = 0;
    h.v[j] = 0.0;
    if (16 * j + gl < n) {
      h.s[j] = slot[e0 + 16 * j + gl];
      h.v[j] = val[e0 + 16 * j + gl];
    }
  }
}

__device__ __forceinline__ double held_dot(const HeldSide &h, const double *xs, const int32_t *__restrict__ slot,
                                           const double *__restrict__ val) {
  const int gl = threadIdx.x & 15;
  double d = 0.0;
#pragma unroll
  for (int j = 0; j < kApplyHeld; j++) {
    const double x = xs[h.s[j]];  // without an entry: slot 0, whose x may be infinite
    d = fma(h.v[j], 16 * j + gl < h.n ? x : 0.0, d);
  }
  for (int e = 16 * kApplyHeld + gl; e < h.n; e += 16) d = fma(val[h.e0 + e], xs[slot[h.e0 + e]], d);
  return group_sum(d);
}

__device__ __forceinline__ void held_add(const HeldSide &h, double c, double *ys, const int32_t *__restrict__ slot,
                                         const double *__restrict__ val) {
  const int gl = threadIdx.x & 15;
#pragma unroll
  for (int j = 0; j < kApplyHeld; j++)
    if (16 * j + gl < h.n) atomicAdd(&ys[h.s[j]], c * h.v[j]);
  for (int e = 16 * kApplyHeld + gl; e < h.n; e += 16) atomicAdd(&ys[slot[h.e0 + e]], c * val[h.e0 + e]);
}

__global__ void __launch_bounds__(64 * kApplyWaves) k_tube_apply(ApplyArgs a) {
  extern __shared__ double lds[];
  double be = 0.0;
  if (a.cg.st) {
    if (cg_ended(a.cg, be, lds, blockIdx.x == 0)) return;
    __syncthreads();  // the sums' LDS is free
  }
  const int4 it = a.items[blockIdx.x];
  const int64_t u0 = a.u_off[it.x];
  const int U = (int)(a.u_off[it.x + 1] - u0);
  const int wave = threadIdx.x >> 6, grp = threadIdx.x >> 4;
  double *xs = lds, *ys = lds + (int64_t)(1 + wave) * a.max_u;
  for (int j = threadIdx.x; j < U; j += blockDim.x) {
    xs[j] = cg_entry(a.cg, be, a.x, a.tube_u[u0 + j]);
#pragma unroll
    for (int v = 0; v < kApplyWaves; v++) lds[(int64_t)(1 + v) * a.max_u + j] = 0.0;
  }
  __syncthreads();
  // group g of the 16 takes pairs from its sixteenth of the segment
  const int len = it.z - it.y, per = (len + 4 * kApplyWaves - 1) / (4 * kApplyWaves);
  const int b = it.y + grp * per, e = b + per < it.z ? b + per : it.z;
  HeldSide l, r, ln, rn;
  double w = 0.0, wn = 0.0;
  auto load = [&](int k, HeldSide &hl, HeldSide &hr, double &ww) {
    int4 m = make_int4(0, 0, 0, 0);
    ww = 0.0;
    if (k < e) {
      m = a.pm[k];
      ww = a.pw[k];
    }
    held_load(hl, m.x, pair_nl(m), a.ent_slot, a.ent_val);
    held_load(hr, m.y, pair_nr(m), a.ent_slot, a.ent_val);
  };
  load(b, l, r, w);
  for (int k = 0; k < per; k++) {
    load(b + k + 1, ln, rn, wn);
    const double dl = held_dot(l, xs, a.ent_slot, a.ent_val), dr = held_dot(r, xs, a.ent_slot, a.ent_val);
    held_add(l, w * dr, ys, a.ent_slot, a.ent_val);
    held_add(r, w * dl, ys, a.ent_slot, a.ent_val);
    l = ln;
    r = rn;
    w = wn;
  }
  __syncthreads();
  const int axis = (int)((unsigned)a.pm[it.y].w >> 30);  // a tube's pairs share one axis
  const double kc = axis == 0 ? a.KC0 : (axis == 1 ? a.KC1 : a.KC2);
  double *out = a.part + a.seg_off[it.x] + (int64_t)it.w * U;
  for (int j = threadIdx.x; j < U; j += blockDim.x) {
    double s = 0.0;
#pragma unroll
    for (int v = 0; v < kApplyWaves; v++) s += lds[(int64_t)(1 + v) * a.max_u + j];
    out[j] = kc * s;
  }
}

// The diagonal of K in the same way: K_jj = sum_i K_i c_alpha sum_g 2 w_g
// L_gi(j) R_gi(j).  A wavefront takes one pair at a time: l summed per node into
// its LDS row, then every entry of r at node j adds 2 w r L(j) to the part.
__global__ void k_tube_diag(ApplyArgs a) {
  extern __shared__ double lds[];
  const int4 it = a.items[blockIdx.x];
  const int64_t u0 = a.u_off[it.x];
  const int U = (int)(a.u_off[it.x + 1] - u0);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  double *ls = lds + (int64_t)wave * a.max_u, *ys = lds + (int64_t)(nw + wave) * a.max_u;
  for (int j = lane; j < U; j += 64) ls[j] = ys[j] = 0.0;
  wave_lds_sync();
  for (int k = it.y + wave; k < it.z; k += nw) {
    const int4 m = a.pm[k];
    const int nl = pair_nl(m), nr = pair_nr(m);
    const double w2 = 2.0 * a.pw[k];
    for (int e = lane; e < nl; e += 64) atomicAdd(&ls[a.ent_slot[m.x + e]], a.ent_val[m.x + e]);
    wave_lds_sync();
    for (int e = lane; e < nr; e += 64) {
      const int s = a.ent_slot[m.y + e];
      const double v = ls[s];
      if (v != 0.0) atomicAdd(&ys[s], w2 * a.ent_val[m.y + e] * v);
    }
    wave_lds_sync();
    for (int e = lane; e < nl; e += 64) ls[a.ent_slot[m.x + e]] = 0.0;
    wave_lds_sync();
  }
  __syncthreads();
  const int axis = (int)((unsigned)a.pm[it.y].w >> 30);
  const double kc = axis == 0 ? a.KC0 : (axis == 1 ? a.KC1 : a.KC2);
  double *out = a.part + a.seg_off[it.x] + (int64_t)it.w * U;
  for (int j = threadIdx.x; j < U; j += blockDim.x) {
    double s = 0.0;
    for (int v = 0; v < nw; v++) s += lds[(int64_t)(nw + v) * a.max_u + j];
    out[j] = kc * s;
  }
}

// y_j = the sum of node j's places in the segments' parts; one wavefront per
// node, four nodes per workgroup and step.  As a step of the conjugate gradients
// it also leaves the direction and its part of its product with y.
__global__ void __launch_bounds__(256) k_tube_sum(const int64_t *__restrict__ row_off, const int2 *__restrict__ row_ts,
                                                  const int64_t *__restrict__ u_off,
                                                  const int64_t *__restrict__ seg_off,
                                                  const double *__restrict__ part, int64_t ndof,
                                                  double *__restrict__ y, const double *__restrict__ x, CgStep c) {
  __shared__ double red[4];
  if (c.st && cg_over(c.st, 2 * (int64_t)c.it + 1)) return;
  const double be = c.st ? c.st->be : 0.0;  // by k_tube_apply
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double xy = 0.0;
  for (int64_t j = (int64_t)blockIdx.x * 4 + wave; j < ndof; j += (int64_t)gridDim.x * 4) {
    double s = 0.0;
    for (int64_t p = row_off[j] + lane; p < row_off[j + 1]; p += 64) {
      const int2 ts = row_ts[p];
      const int64_t U = u_off[ts.x + 1] - u_off[ts.x], e = seg_off[ts.x + 1];
      for (int64_t o = seg_off[ts.x] + ts.y; o < e; o += U) s += part[o];
    }
    for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o, 64);
    if (lane == 0) {
      y[j] = s;
      if (c.st) {
        const double pj = cg_entry(c, be, x, j);
        c.pn[j] = pj;
        xy = fma(s, pj, xy);
      }
    }
  }
  if (!c.st) return;
  if (lane == 0) red[wave] = xy;
  __syncthreads();
  if (threadIdx.x == 0) c.dot[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

struct TubeMfmaArgs {
  const int64_t *tube_off;
  const int4 *pm;
  const double *pw;
  const int64_t *mk_pair;
  const uint32_t *mk_meta;
  const float *mk_val;
  const int64_t *blk_off;
  double *blk;
  double KC0, KC1, KC2;
};

// One merged entry into the operand panels of buffer `b`: row slot - rx0
// of X (column c, W_p v) and row slot - ry0 of Y (column c ^ 1, v), each
// as hi and lo.
__device__ __forceinline__ void tube_put(TubeMfmaSmem &sm, int b, uint32_t mt, float v, const float *wv, float ysc,
                                         int rx0, int ry0) {
  const int sl = (int)(mt & 0xffffu), c = (int)(mt >> 16);
  const int rx = sl - rx0, ry = sl - ry0;
  if ((unsigned)rx < (unsigned)kRegion) {
    const float x = wv[c >> 1] * v;
    const _Float16 h = (_Float16)x;
    const int g = tswz(rx, c >> 3);
    ((_Float16 *)&sm.hx[b][0][rx][g])[c & 7] = h;
    ((_Float16 *)&sm.hx[b][1][rx][g])[c & 7] = (_Float16)(x - (float)h);
  }
  if ((unsigned)ry < (unsigned)kRegion) {
    const float y = v * ysc;
    const _Float16 h = (_Float16)y;
    const int cy = c ^ 1;
    const int g = tswz(ry, cy >> 3);
    ((_Float16 *)&sm.hy[b][0][ry][g])[cy & 7] = h;
    ((_Float16 *)&sm.hy[b][1][ry][g])[cy & 7] = (_Float16)(y - (float)h);
  }
}

// Work item b = blockIdx.x of n_items (the grid); items {-1, ..} pad the
// per-XCD lists and exit.
__global__ void __launch_bounds__(kTubeThreads) k_tube_mfma(TubeMfmaArgs a, const int4 *__restrict__ items, int64_t n_items,
                                                   const int2 *__restrict__ texp) {
  __shared__ TubeMfmaSmem sm;
  __shared__ float sw[2][kChunkPairs];  // W_p 2^-ex of the chunk's pairs (double-buffered)
  const int64_t bw = blockIdx.x;
  if (bw >= n_items) return;
  const int4 it = items[bw];
  if (it.x < 0) return;
  const int64_t T = it.x;
  const int U = it.w, rx0 = kRegion * it.y, ry0 = kRegion * it.z;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6, wr = w >> 2, wc = w & 3;
  const int64_t *__restrict__ mk_pair = a.mk_pair;
  const uint32_t *__restrict__ mk_meta = a.mk_meta;
  const float *__restrict__ mk_val = a.mk_val;
  const double *__restrict__ pw = a.pw;
  const int64_t k0 = a.tube_off[T], k1 = a.tube_off[T + 1];
  const int2 te0 = texp[T];
  const int2 te = make_int2(tube_scale_exp(te0.x), tube_scale_exp(te0.y));
  // the tube's pairs share one axis, so one coefficient
  const int axis = k1 > k0 ? (int)((unsigned)a.pm[k0].w >> 30) : 0;
  const double xsc = (axis == 0 ? a.KC0 : (axis == 1 ? a.KC1 : a.KC2)) * ldexp(1.0, -te.x);
  const float ysc = ldexpf(1.f, -te.y);
  // both panel buffers start at zero; a clear is 2 x 16 bytes per thread
  // of the buffer's hx and of its hy (16 KB each), consecutive lanes on
  // consecutive 16-byte slots
  const half8 z8 = {0, 0, 0, 0, 0, 0, 0, 0};
  auto clear = [&](int b) {
    half8 *px = &sm.hx[b][0][0][0], *py = &sm.hy[b][0][0][0];
#pragma unroll
    for (int j = 0; j < 1024 / kTubeThreads; j++) {
      px[t + kTubeThreads * j] = z8;
      py[t + kTubeThreads * j] = z8;
    }
  };
  clear(0);
  clear(1);
  f32x4v acc[4][2];
#pragma unroll
  for (int x = 0; x < 4; x++)
#pragma unroll
    for (int y = 0; y < 2; y++) acc[x][y] = f32x4v{0.f, 0.f, 0.f, 0.f};
  const int q = lane >> 4;
  // A chunk's merged entries are one contiguous range [e0, e1); thread t
  // takes e0 + t + kTubeThreads j.  Loads run ahead of their use: while chunk c is
  // scattered and multiplied, the entries of chunks c + 1 and c + 2, the
  // bounds of chunk c + 3 and the pair weights of chunk c + 2 are in flight.
  constexpr int kPre = 4;
  uint32_t cm[kPre], nm[kPre], fm[kPre];
  float cv[kPre], nv[kPre], fv[kPre];
  auto bounds = [&](int64_t kc, int64_t &b0, int64_t &b1) {
    if (kc < k1) {
      b0 = mk_pair[kc];
      b1 = mk_pair[kc + kChunkPairs < k1 ? kc + kChunkPairs : k1];
    } else {
      b0 = b1 = 0;
    }
  };
  auto entries = [&](int64_t b0, int64_t b1, uint32_t(&em)[kPre], float(&ev)[kPre]) {
#pragma unroll
    for (int j = 0; j < kPre; j++) {
      const int64_t i = b0 + t + kTubeThreads * j;
      const int64_t ic = i < b1 ? i : b0;
      em[j] = b1 > b0 ? mk_meta[ic] : 0u;
      ev[j] = b1 > b0 ? mk_val[ic] : 0.f;
    }
  };
  auto weight = [&](int64_t kc) { return t < kChunkPairs && kc + t < k1 ? (float)(pw[kc + t] * xsc) : 0.f; };
  // bounds of chunks c, c + 1, c + 2 (c = the current chunk)
  int64_t c0, c1, n0, n1, f0, f1;
  bounds(k0, c0, c1);
  bounds(k0 + kChunkPairs, n0, n1);
  bounds(k0 + 2 * kChunkPairs, f0, f1);
  entries(c0, c1, cm, cv);
  entries(n0, n1, nm, nv);
  if (t < kChunkPairs) sw[0][t] = weight(k0);
  float wnext = weight(k0 + kChunkPairs);
  int buf = 0;
  for (int64_t kc = k0; kc < k1; kc += kChunkPairs) {
    // issued now, used two iterations later: the entries of chunk c + 2;
    // one iteration later: the bounds of chunk c + 3, the weights of c + 2
    entries(f0, f1, fm, fv);
    int64_t g0, g1;
    bounds(kc + 3 * kChunkPairs, g0, g1);
    const float wfar = weight(kc + 2 * kChunkPairs);
    // buffer buf ^ 1 was read by the previous chunk's products, which every
    // wavefront finished before this barrier; buffer buf was cleared during
    // the previous chunk
    __syncthreads();
    clear(buf ^ 1);
#pragma unroll
    for (int j = 0; j < kPre; j++)
      if (c0 + t + kTubeThreads * j < c1) tube_put(sm, buf, cm[j], cv[j], sw[buf], ysc, rx0, ry0);
    for (int64_t i = c0 + t + kTubeThreads * kPre; i < c1; i += kTubeThreads) tube_put(sm, buf, mk_meta[i], mk_val[i], sw[buf], ysc, rx0, ry0);
    if (t < kChunkPairs) sw[buf ^ 1][t] = wnext;
    __syncthreads();
    half8 ah[4], al[4], bh[2], bl[2];
#pragma unroll
    for (int x = 0; x < 4; x++) {
      const int ar = 64 * wr + 16 * x + (lane & 15);
      ah[x] = sm.hx[buf][0][ar][tswz(ar, q)];
      al[x] = sm.hx[buf][1][ar][tswz(ar, q)];
    }
#pragma unroll
    for (int y = 0; y < 2; y++) {
      const int br = 32 * wc + 16 * y + (lane & 15);
      bh[y] = sm.hy[buf][0][br][tswz(br, q)];
      bl[y] = sm.hy[buf][1][br][tswz(br, q)];
    }
#pragma unroll
    for (int x = 0; x < 4; x++)
#pragma unroll
      for (int y = 0; y < 2; y++) {
        acc[x][y] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah[x], bh[y], acc[x][y], 0, 0, 0);
        acc[x][y] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah[x], bl[y], acc[x][y], 0, 0, 0);
        acc[x][y] = __builtin_amdgcn_mfma_f32_16x16x32_f16(al[x], bh[y], acc[x][y], 0, 0, 0);
      }
    buf ^= 1;
#pragma unroll
    for (int j = 0; j < kPre; j++) {
      cm[j] = nm[j];
      cv[j] = nv[j];
      nm[j] = fm[j];
      nv[j] = fv[j];
    }
    c0 = n0;
    c1 = n1;
    n0 = f0;
    n1 = f1;
    f0 = g0;
    f1 = g1;
    wnext = wfar;
  }
  // region (I, J) of the block and, off the diagonal of regions, its mirror
  double *out = a.blk + a.blk_off[T];
  const int eu = te.x + te.y;
#pragma unroll
  for (int x = 0; x < 4; x++)
#pragma unroll
    for (int y = 0; y < 2; y++)
#pragma unroll
      for (int i = 0; i < 4; i++) {
        const int r = rx0 + 64 * wr + 16 * x + 4 * (lane >> 4) + i;
        const int c = ry0 + 32 * wc + 16 * y + (lane & 15);
        if (r < U && c < U) {
          const double v = ldexp((double)acc[x][y][i], eu);
          out[(int64_t)r * U + c] = v;
          if (it.y != it.z) out[(int64_t)c * U + r] = v;
        }
      }
}

}  // namespace

void free_tubes(TubePlan &tp) {
  dfree(tp.pair_sorted); dfree(tp.pm); dfree(tp.pw); dfree(tp.tube_off); dfree(tp.u_off); dfree(tp.tube_u); dfree(tp.ent_slot);
  dfree(tp.row_off); dfree(tp.row_ts); dfree(tp.items); dfree(tp.fitems); dfree(tp.blk_off); dfree(tp.blk);
  dfree(tp.mitems); dfree(tp.texp);
  dfree(tp.mk_pair); dfree(tp.mk_meta); dfree(tp.mk_val); dfree(tp.mg_idx); dfree(tp.pk_tube);
  dfree(tp.cstart);
  dfree(tp.aitems); dfree(tp.seg_off); dfree(tp.part);
  tp = TubePlan();
}

int build_tubes(fpde_mesh *m, Plan &P, const TubeGeom &q, double kappa, hipStream_t s) {
  TubePlan &tp = P.tubes;
  free_tubes(tp);
  if (m->ndof == 0 || P.G == 0) return FPDE_OK;
  const int dim = q.dim;
  const int64_t n = dim * P.G;
  if (n >= (int64_t(1) << 31)) return FPDE_EUNSUPPORTED;
  // cell size from the mean element size (edge of the regular simplex of mean
  // volume), stretched along each axis as the mean edge is, over up to 4096 elements.
  // With square cells 8 x 100 x 100 cells 20 times as long as thin had tubes of 1 756
  // nodes instead of 792, and took 219 against 116 ms (Riesz matrix) and 11.0 against
  // 4.9 ms (a product).
  std::vector<double> xyz(dim * q.nv), vol(q.nt);
  std::vector<int32_t> elem((dim + 1) * q.nt);
  FPDE_HIP(hipMemcpyAsync(xyz.data(), q.xyz, sizeof(double) * dim * q.nv, hipMemcpyDeviceToHost, s));
  FPDE_HIP(hipMemcpyAsync(vol.data(), q.vol, sizeof(double) * q.nt, hipMemcpyDeviceToHost, s));
  FPDE_HIP(hipMemcpyAsync(elem.data(), q.elem, sizeof(int32_t) * (dim + 1) * q.nt, hipMemcpyDeviceToHost, s));
  FPDE_HIP(hipStreamSynchronize(s));
  double lo[3] = {1e300, 1e300, 1e300}, hi[3] = {-1e300, -1e300, -1e300}, V = 0.0;
  for (int64_t v = 0; v < q.nv; v++)
    for (int d = 0; d < dim; d++) {
      lo[d] = std::min(lo[d], xyz[dim * v + d]);
      hi[d] = std::max(hi[d], xyz[dim * v + d]);
    }
  for (double x : vol) V += x;
  double edge[3] = {0.0, 0.0, 0.0}, mean = 1.0;
  for (int64_t t = 0; t < q.nt; t += (q.nt + 4095) / 4096)
    for (int a = 0; a < dim; a++)
      for (int b = a + 1; b <= dim; b++)
        for (int d = 0; d < dim; d++)
          edge[d] += std::fabs(xyz[dim * (int64_t)elem[(dim + 1) * t + a] + d] -
                               xyz[dim * (int64_t)elem[(dim + 1) * t + b] + d]);
  for (int d = 0; d < dim; d++) mean *= std::pow(edge[d], 1.0 / dim);
  const double h = dim == 3 ? std::cbrt(6.0 * std::sqrt(2.0) * V / (double)q.nt)
                            : std::sqrt(4.0 / std::sqrt(3.0) * V / (double)q.nt);
  TubeCells cells{};
  for (int d = 0; d < dim; d++) {
    const double c = kappa * h * edge[d] / mean, n = std::ceil((hi[d] - lo[d]) / c) + 1.0;
    if (!(n < 2147483648.0)) return FPDE_EUNSUPPORTED;
    cells.lo[d] = lo[d];
    cells.inv_c[d] = 1.0 / c;
    cells.n[d] = (int)n;
  }
  double per_axis = 0.0;
  for (int i = 0; i < dim; i++) {
    double n = 1.0;
    for (int d = 1; d < dim; d++) n *= cells.n[(i + d) % dim];
    per_axis = std::max(per_axis, n);
  }
  if (dim * per_axis >= 4294967295.0) return FPDE_EUNSUPPORTED;
  cells.per_axis = (uint32_t)per_axis;

  uint32_t *key = nullptr, *key2 = nullptr;
  int32_t *val = nullptr, *head = nullptr, *tid = nullptr;
  int64_t *u_cnt = nullptr, *row_cnt = nullptr, *cursor = nullptr, *usq = nullptr;
  void *tmp = nullptr;
  size_t tmp_bytes = 0;
  auto cleanup = [&]() {
    dfree(key); dfree(key2); dfree(val); dfree(head); dfree(tid);
    dfree(u_cnt); dfree(row_cnt); dfree(cursor); dfree(usq);
    if (tmp) (void)hipFree(tmp);
    tmp = nullptr;
  };
  auto fail = [&](int code) {
    cleanup();
    free_tubes(tp);
    return code;
  };
  auto scratch = [&](size_t need) -> int {
    if (need <= tmp_bytes) return FPDE_OK;
    if (tmp) (void)hipFree(tmp);
    tmp = nullptr;
    tmp_bytes = 0;
    if (hipMalloc(&tmp, need) != hipSuccess) return FPDE_ENOMEM;
    tmp_bytes = need;
    return FPDE_OK;
  };
#define TRY_T(x)                          \
  do {                                    \
    int st_ = (x);                        \
    if (st_ != FPDE_OK) return fail(st_); \
  } while (0)
#define HIP_T(x)                                     \
  do {                                               \
    if ((x) != hipSuccess) return fail(FPDE_EHIP);   \
  } while (0)
  int st;
  TRY_T(dalloc(&key, n));
  TRY_T(dalloc(&key2, n));
  TRY_T(dalloc(&val, n));
  TRY_T(dalloc(&tp.pair_sorted, n));
  k_pair_keys<<<nblocks(n), 256, 0, s>>>(q, P.nq, P.G, cells, key, val);
  size_t need = 0;
  const int end_bit = 32;
  HIP_T(hipcub::DeviceRadixSort::SortPairs(nullptr, need, key, key2, val, tp.pair_sorted, (int)n, 0, end_bit, s));
  TRY_T(scratch(need));
  HIP_T(hipcub::DeviceRadixSort::SortPairs(tmp, tmp_bytes, key, key2, val, tp.pair_sorted, (int)n, 0, end_bit, s));
  TRY_T(dalloc(&head, n));
  TRY_T(dalloc(&tid, n));
  k_heads<<<nblocks(n), 256, 0, s>>>(key2, n, head);
  HIP_T(hipcub::DeviceScan::ExclusiveSum(nullptr, need, head, tid, (int)n, s));
  TRY_T(scratch(need));
  HIP_T(hipcub::DeviceScan::ExclusiveSum(tmp, tmp_bytes, head, tid, (int)n, s));
  int32_t last_tid = 0, last_head = 0;
  HIP_T(hipMemcpyAsync(&last_tid, tid + n - 1, sizeof(int32_t), hipMemcpyDeviceToHost, s));
  HIP_T(hipMemcpyAsync(&last_head, head + n - 1, sizeof(int32_t), hipMemcpyDeviceToHost, s));
  HIP_T(hipStreamSynchronize(s));
  tp.n_tubes = (int64_t)last_tid + last_head;
  const int64_t nT = tp.n_tubes;
  TRY_T(dalloc(&tp.tube_off, nT + 1));
  k_tube_off<<<nblocks(n), 256, 0, s>>>(head, tid, n, tp.tube_off);
  TRY_T(dalloc(&tp.pm, n));
  TRY_T(dalloc(&tp.pw, n));
  k_pair_meta<<<nblocks(n), 256, 0, s>>>(tp.pair_sorted, n, P.G, P.nq, P.off, q.rule + (dim + 1) * P.nq, q.vol, tp.pm,
                                         tp.pw);
  dfree(key); dfree(key2); dfree(val); dfree(head); dfree(tid);

  // node sets
  TRY_T(dalloc(&u_cnt, nT + 1));
  TRY_T(dalloc(&tp.u_off, nT + 1));
  HIP_T(hipMemsetAsync(u_cnt, 0, sizeof(int64_t) * (nT + 1), s));
  k_tube_count<<<(unsigned)nT, kPlanThreads, 0, s>>>(tp.tube_off, tp.pm, P.ent_dof, u_cnt, m->flag);
  int f = take_flag(m, s);
  if (f != 0) return fail(f < 0 ? f : FPDE_EHIP);
  HIP_T(hipcub::DeviceScan::ExclusiveSum(nullptr, need, u_cnt, tp.u_off, (int)(nT + 1), s));
  TRY_T(scratch(need));
  HIP_T(hipcub::DeviceScan::ExclusiveSum(tmp, tmp_bytes, u_cnt, tp.u_off, (int)(nT + 1), s));
  HIP_T(hipMemcpyAsync(&tp.n_u, tp.u_off + nT, sizeof(int64_t), hipMemcpyDeviceToHost, s));
  HIP_T(hipStreamSynchronize(s));
  TRY_T(dalloc(&tp.tube_u, tp.n_u));
  TRY_T(dalloc(&tp.ent_slot, P.n_ent));
  TRY_T(dalloc(&row_cnt, m->ndof + 1));
  HIP_T(hipMemsetAsync(row_cnt, 0, sizeof(int64_t) * (m->ndof + 1), s));
  k_tube_fill<<<(unsigned)nT, kPlanThreads, 0, s>>>(tp.tube_off, tp.pm, P.ent_dof, tp.u_off, tp.tube_u, tp.ent_slot, row_cnt);
  TRY_T(dalloc(&tp.row_off, m->ndof + 1));
  HIP_T(hipcub::DeviceScan::ExclusiveSum(nullptr, need, row_cnt, tp.row_off, (int)(m->ndof + 1), s));
  TRY_T(scratch(need));
  HIP_T(hipcub::DeviceScan::ExclusiveSum(tmp, tmp_bytes, row_cnt, tp.row_off, (int)(m->ndof + 1), s));
  TRY_T(dalloc(&cursor, m->ndof + 1));
  HIP_T(hipMemcpyAsync(cursor, tp.row_off, sizeof(int64_t) * (m->ndof + 1), hipMemcpyDeviceToDevice, s));
  TRY_T(dalloc(&tp.row_ts, tp.n_u));
  k_row_places<<<(unsigned)nT, 256, 0, s>>>(tp.u_off, nT, tp.tube_u, cursor, tp.row_ts);

  // block offsets, then the pass-1 work items {tube, first block row, rows, |U_T|}
  TRY_T(dalloc(&usq, nT + 1));
  TRY_T(dalloc(&tp.blk_off, nT + 1));
  HIP_T(hipMemsetAsync(usq, 0, sizeof(int64_t) * (nT + 1), s));
  k_block_sizes<<<nblocks(nT), 256, 0, s>>>(tp.u_off, nT, usq);
  HIP_T(hipcub::DeviceScan::ExclusiveSum(nullptr, need, usq, tp.blk_off, (int)(nT + 1), s));
  TRY_T(scratch(need));
  HIP_T(hipcub::DeviceScan::ExclusiveSum(tmp, tmp_bytes, usq, tp.blk_off, (int)(nT + 1), s));
  std::vector<int64_t> uo(nT + 1), to(nT + 1);
  HIP_T(hipMemcpyAsync(&tp.blk_n, tp.blk_off + nT, sizeof(int64_t), hipMemcpyDeviceToHost, s));
  HIP_T(hipMemcpyAsync(uo.data(), tp.u_off, sizeof(int64_t) * (nT + 1), hipMemcpyDeviceToHost, s));
  HIP_T(hipMemcpyAsync(to.data(), tp.tube_off, sizeof(int64_t) * (nT + 1), hipMemcpyDeviceToHost, s));
  HIP_T(hipStreamSynchronize(s));
  {
    tp.max_u = 0;
    for (int64_t T = 0; T < nT; T++) tp.max_u = std::max<int64_t>(tp.max_u, uo[T + 1] - uo[T]);
    // largest tubes first (by pairs times nodes), so that none starts last
    std::vector<int64_t> order(nT);
    for (int64_t T = 0; T < nT; T++) order[T] = T;
    std::stable_sort(order.begin(), order.end(), [&](int64_t x, int64_t y) {
      return (to[x + 1] - to[x]) * (uo[x + 1] - uo[x]) > (to[y + 1] - to[y]) * (uo[y + 1] - uo[y]);
    });
    double work = 0.0;
    auto weight = [&](int64_t T) {
      const double U = (double)(uo[T + 1] - uo[T]);
      return (double)(to[T + 1] - to[T]) * U * U;
    };
    for (int64_t T = 0; T < nT; T++) work += weight(T);
    std::vector<int4> items, fitems;
    for (const int64_t T : order) {
      const int U = (int)(uo[T + 1] - uo[T]);
      if (U == 0) continue;
      const int64_t bands = ((int64_t)U * (U + 1) / 2 + kBand - 1) / kBand;
      const double share = U <= kSplitFrom ? 0.0 : weight(T) * kShares / work;
      const int parts = std::max(1, (int)share);
      const int R = std::min({U, kBand / band_stride(U), std::max(kMinRows, (U + parts - 1) / parts)});
      for (int r0 = 0; r0 < U; r0 += R) fitems.push_back(make_int4((int)T, r0, std::min(R, U - r0), U));
      const bool full = bands > kTriBands || (bands > 1 && share >= 1.0) || share >= 4.0;
      for (int r0 = 0; r0 < U;) {
        const int r = full ? std::min(R, U - r0) : band_rows(U, r0, kBand);
        items.push_back(make_int4((int)T, r0, full ? r | kFullRows : r, U));
        r0 += r;
      }
    }
    auto upload = [&](const std::vector<int4> &v, int4 **p, int64_t *count) -> int {
      *count = (int64_t)v.size();
      FPDE_TRY(dalloc(p, v.size()));
      if (!v.empty()) FPDE_HIP(hipMemcpyAsync(*p, v.data(), sizeof(int4) * v.size(), hipMemcpyHostToDevice, s));
      FPDE_HIP(hipStreamSynchronize(s));
      return FPDE_OK;
    };
    TRY_T(upload(items, &tp.items, &tp.n_items));
    TRY_T(upload(fitems, &tp.fitems, &tp.n_fitems));
  }
  // Segments of the matrix-free product: at most kSegMax pairs, fewer on small
  // meshes so that there are a few thousand, in multiples of the 16 groups of
  // a workgroup.
  {
    constexpr int64_t kSegMin = 32, kSegMax = 512;
    const int64_t seg = std::min(kSegMax, std::max(kSegMin, n / 4096 / 16 * 16));
    std::vector<int64_t> so(nT + 1);
    std::vector<int4> items;
    int64_t off = 0;
    for (int64_t T = 0; T < nT; T++) {
      so[T] = off;
      if (uo[T + 1] == uo[T]) continue;
      int q = 0;
      for (int64_t k = to[T]; k < to[T + 1]; k += seg, q++)
        items.push_back(make_int4((int)T, (int)k, (int)std::min(k + seg, to[T + 1]), q));
      off += q * (uo[T + 1] - uo[T]);
    }
    so[nT] = off;
    tp.n_part = off;
    tp.n_aitems = (int64_t)items.size();
    TRY_T(dalloc(&tp.seg_off, nT + 1));
    TRY_T(dalloc(&tp.aitems, items.size() > 0 ? items.size() : 1));
    HIP_T(hipMemcpyAsync(tp.seg_off, so.data(), sizeof(int64_t) * (nT + 1), hipMemcpyHostToDevice, s));
    if (!items.empty())
      HIP_T(hipMemcpyAsync(tp.aitems, items.data(), sizeof(int4) * items.size(), hipMemcpyHostToDevice, s));
    HIP_T(hipStreamSynchronize(s));
  }
  HIP_T(hipGetLastError());
  f = take_flag(m, s);
  if (f != 0) return fail(f < 0 ? f : FPDE_EHIP);
  cleanup();
  return FPDE_OK;
#undef TRY_T
#undef HIP_T
}

// Plan of the matrix-core contraction: work items over the upper 128 x 128
// regions of every tube block, and the merge structure of every pair (merged
// index per entry, slot and inner column per merged entry).  Tubes larger
// than kMergeSlots or pairs with more than kMergeMax merged entries leave
// mfma_ok false (the FP64 accumulation then serves the mixed path).
static int build_mfma_plan(fpde_mesh *m, Plan &P, TubePlan &tp, hipStream_t s) {
  const int64_t nT = tp.n_tubes, nP = 3 * P.G;
  tp.mfma_ok = false;
  if (nT == 0 || tp.max_u > kMergeSlots) return FPDE_OK;
  int64_t *pcnt = nullptr;
  int *maxc = nullptr;
  void *tmp = nullptr;
  size_t need = 0, have = 0;
  int st = FPDE_OK;
  auto done = [&](int code) {
    dfree(pcnt);
    dfree(maxc);
    if (tmp) (void)hipFree(tmp);
    return code;
  };
  auto scan = [&](const int64_t *in, int64_t *out, int64_t n) {
    if (hipcub::DeviceScan::ExclusiveSum(nullptr, need, in, out, (int)n, s) != hipSuccess) return FPDE_EHIP;
    if (need > have) {
      if (tmp) (void)hipFree(tmp);
      tmp = nullptr;
      if (hipMalloc(&tmp, need) != hipSuccess) return FPDE_ENOMEM;
      have = need;
    }
    return hipcub::DeviceScan::ExclusiveSum(tmp, need, in, out, (int)n, s) == hipSuccess ? FPDE_OK : FPDE_EHIP;
  };
  auto to_host = [&](const void *src, void *dst, size_t bytes) {
    return hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, s) == hipSuccess &&
           hipStreamSynchronize(s) == hipSuccess;
  };
  // merged entries per pair, scanned
  if ((st = dalloc(&pcnt, nP + 1)) != FPDE_OK) return done(st);
  if ((st = dalloc(&maxc, 1)) != FPDE_OK) return done(st);
  if (hipMemsetAsync(pcnt, 0, sizeof(int64_t) * (nP + 1), s) != hipSuccess) return done(FPDE_EHIP);
  if (hipMemsetAsync(maxc, 0, sizeof(int), s) != hipSuccess) return done(FPDE_EHIP);
  k_merge_pairs<false><<<(unsigned)nP, 64, 0, s>>>(tp.tube_off, nT, tp.pm, nP, tp.ent_slot, pcnt, nullptr, nullptr,
                                                    nullptr, nullptr, maxc);
  int mc = 0;
  if (!to_host(maxc, &mc, sizeof(int))) return done(FPDE_EHIP);
  if (mc > kMergeMax) return done(FPDE_OK);
  if ((st = dalloc(&tp.mk_pair, nP + 1)) != FPDE_OK) return done(st);
  if ((st = scan(pcnt, tp.mk_pair, nP + 1)) != FPDE_OK) return done(st);
  int64_t n_mk = 0;
  if (!to_host(tp.mk_pair + nP, &n_mk, sizeof(int64_t))) return done(FPDE_EHIP);
  if ((st = dalloc(&tp.mk_meta, n_mk > 0 ? n_mk : 1)) != FPDE_OK) return done(st);
  if ((st = dalloc(&tp.mk_val, n_mk > 0 ? n_mk : 1)) != FPDE_OK) return done(st);
  if ((st = dalloc(&tp.mg_idx, P.n_ent > 0 ? P.n_ent : 1)) != FPDE_OK) return done(st);
  if ((st = dalloc(&tp.pk_tube, nP > 0 ? nP : 1)) != FPDE_OK) return done(st);
  k_merge_pairs<true><<<(unsigned)nP, 64, 0, s>>>(tp.tube_off, nT, tp.pm, nP, tp.ent_slot, nullptr, tp.mk_pair,
                                                   tp.mg_idx, tp.mk_meta, tp.pk_tube, nullptr);
  // Region work items, balanced over the eight XCDs (the hardware deals
  // workgroup b to XCD b mod 8): whole tubes, largest cost first, each to
  // the XCD with the least work so far (cost = regions x chunks of 16
  // pairs); the items of XCD x at positions 8 j + x in tube order, padded
  // with {-1} at the end.  A tube's regions stay on one XCD, whose L2 then
  // serves its merged entries to all of them.
  std::vector<int64_t> toff(nT + 1), uoff(nT + 1);
  if (!to_host(tp.tube_off, toff.data(), sizeof(int64_t) * (nT + 1))) return done(FPDE_EHIP);
  if (!to_host(tp.u_off, uoff.data(), sizeof(int64_t) * (nT + 1))) return done(FPDE_EHIP);
  std::vector<int64_t> cost(nT), order(nT);
  for (int64_t T = 0; T < nT; T++) {
    const int64_t nr = (uoff[T + 1] - uoff[T] + kRegion - 1) / kRegion;
    const int64_t chunks = (toff[T + 1] - toff[T] + kChunkPairs - 1) / kChunkPairs;
    cost[T] = nr * (nr + 1) / 2 * (chunks + 1);
    order[T] = T;
  }
  std::stable_sort(order.begin(), order.end(), [&](int64_t x, int64_t y) { return cost[x] > cost[y]; });
  std::vector<int4> lists[8];
  int64_t load[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  for (const int64_t T : order) {
    const int x = (int)(std::min_element(load, load + 8) - load);
    load[x] += cost[T];
    const int U = (int)(uoff[T + 1] - uoff[T]);
    const int nr = (U + kRegion - 1) / kRegion;
    for (int I = 0; I < nr; I++)
      for (int J = I; J < nr; J++) lists[x].push_back(make_int4((int)T, I, J, U));
  }
  size_t per = 0;
  for (int x = 0; x < 8; x++) per = std::max(per, lists[x].size());
  if (8 * (int64_t)per >= (int64_t(1) << 31)) return done(FPDE_EUNSUPPORTED);
  std::vector<int4> items(8 * per, make_int4(-1, 0, 0, 0));
  for (int x = 0; x < 8; x++)
    for (size_t j = 0; j < lists[x].size(); j++) items[8 * j + x] = lists[x][j];
  if ((st = dalloc(&tp.mitems, items.size() > 0 ? items.size() : 1)) != FPDE_OK) return done(st);
  if (!items.empty() && (hipMemcpyAsync(tp.mitems, items.data(), sizeof(int4) * items.size(), hipMemcpyHostToDevice,
                                        s) != hipSuccess ||
                         hipStreamSynchronize(s) != hipSuccess))
    return done(FPDE_EHIP);
  tp.n_mitems = (int64_t)items.size();
  if (hipGetLastError() != hipSuccess) return done(FPDE_EHIP);
  tp.mfma_ok = true;
  return done(FPDE_OK);
}

// Pass 1 (the tube blocks) for order p->alpha and coefficients p->K:
// FP64 LDS accumulation, or for the mixed-precision matrix the split-FP16
// matrix-core contraction.
static int accumulate_tube_blocks(fpde_mesh *m, Plan &P, const fpde_params *p, hipStream_t s) {
  TubePlan &tp = P.tubes;
  if (!tp.blk) {
    FPDE_TRY(dalloc(&tp.blk, tp.blk_n > 0 ? tp.blk_n : 1));
  }
  Order o = order_scalars(p->alpha);
  AccumArgs a{};
  a.tube_off = tp.tube_off;
  a.pm = tp.pm;
  a.pw = tp.pw;
  a.items = tp.items;
  a.ent_slot = tp.ent_slot;
  a.ent_val = P.ent_val;
  a.blk_off = tp.blk_off;
  a.blk = tp.blk;
  a.KC0 = p->K[0] * o.c_alpha;
  a.KC1 = p->K[1] * o.c_alpha;
  a.KC2 = p->K[2] * o.c_alpha;
  // split FP16 on the matrix cores for the mixed-precision matrix (planned
  // once: work items and merge structure; merged values and exponents at
  // every assembly, as they follow the values)
  if (p->precision == FPDE_MIXED && !tp.mfma_planned) {
    FPDE_TRY(build_mfma_plan(m, P, tp, s));
    tp.mfma_planned = true;
  }
  if (p->precision == FPDE_MIXED && tp.mfma_ok) {
    if (!tp.texp) FPDE_TRY(dalloc(&tp.texp, tp.n_tubes > 0 ? tp.n_tubes : 1));
    const int64_t nP = 3 * P.G;
    const long ta = timer_begin(m, s, FPDE_STAGE_ACCUM);
    k_fill_int2<<<nblocks(tp.n_tubes), 256, 0, s>>>(tp.texp, tp.n_tubes, make_int2(INT_MIN, INT_MIN));
    // eight workgroups of four wavefronts per CU, each wavefront looping
    const unsigned mgrid = (unsigned)std::min<int64_t>(nblocks(nP, 4), 256 * 8);
    k_merge_vals<<<mgrid, 256, 0, s>>>(tp.pm, tp.pw, tp.mk_pair, tp.pk_tube, tp.mg_idx, nP, P.ent_val, a.KC0, a.KC1,
                                       a.KC2, tp.mk_val, tp.texp);
    if (tp.n_mitems > 0) {
      TubeMfmaArgs ma{tp.tube_off, tp.pm, tp.pw, tp.mk_pair, tp.mk_meta, tp.mk_val, tp.blk_off, tp.blk,
                      a.KC0, a.KC1, a.KC2};
      k_tube_mfma<<<(unsigned)tp.n_mitems, kTubeThreads, 0, s>>>(ma, tp.mitems, tp.n_mitems, tp.texp);
    }
    timer_end(m, FPDE_STAGE_ACCUM, ta, s);
    return FPDE_OK;
  }
  const long ta = timer_begin(m, s, FPDE_STAGE_ACCUM);
  // deterministic: one wavefront per item walks the tube's pairs in order
  if (tp.n_items > 0)
    k_tube_accum<<<(unsigned)tp.n_items, p->deterministic ? 64 : kAccumThreads, sizeof(double) * kBand, s>>>(a);
  timer_end(m, FPDE_STAGE_ACCUM, ta, s);
  return FPDE_OK;
}

// Arguments of the row pass; the chunk starts of every tube are computed
// on first use (and again if the chunk width changes).
static int gather_args(fpde_mesh *m, Plan &P, int64_t lda, hipStream_t s, GatherArgs &gch) {
  TubePlan &tp = P.tubes;
  const int chunk = (int)(m->ndof < 8192 ? m->ndof : 8192);
  const int nch = (int)((m->ndof + chunk - 1) / chunk);
  if (!tp.cstart || tp.cs_chunk != chunk) {
    dfree(tp.cstart);
    tp.cs_chunk = 0;
    const int64_t ncs = tp.n_tubes * (nch + 1);
    FPDE_TRY(dalloc(&tp.cstart, ncs > 0 ? ncs : 1));
    if (ncs > 0) k_chunk_starts<<<nblocks(ncs), 256, 0, s>>>(tp.u_off, tp.tube_u, tp.n_tubes, chunk, nch, tp.cstart);
    FPDE_HIP(hipGetLastError());
    tp.cs_chunk = chunk;
  }
  gch = GatherArgs{};
  gch.row_off = tp.row_off;
  gch.row_ts = tp.row_ts;
  gch.u_off = tp.u_off;
  gch.tube_u = tp.tube_u;
  gch.blk_off = tp.blk_off;
  gch.blk = tp.blk;
  gch.cstart = tp.cstart;
  gch.ndof = m->ndof;
  gch.lda = lda;
  gch.chunk = chunk;
  gch.nch = nch;
  return FPDE_OK;
}

static unsigned gather_grid(int64_t ndof) {
  const int64_t slots = 8 * ((ndof + 7) / 8);
  return (unsigned)(slots < 65536 ? slots : 65536);
}

// y = K x (diag: its diagonal) from the plan's current values
static int apply_tubes(fpde_mesh *m, Plan &P, const fpde_params *p, const double *x, double *y, bool diag,
                       hipStream_t s, const CgStep *cg) {
  TubePlan &tp = P.tubes;
  if (!tp.part) FPDE_TRY(dalloc(&tp.part, (size_t)tp.n_part));
  const Order o = order_scalars(p->alpha);
  ApplyArgs a{};
  a.items = tp.aitems;
  a.pm = tp.pm;
  a.pw = tp.pw;
  a.u_off = tp.u_off;
  a.tube_u = tp.tube_u;
  a.seg_off = tp.seg_off;
  a.ent_slot = tp.ent_slot;
  a.ent_val = P.ent_val;
  a.x = x;
  a.part = tp.part;
  a.KC0 = p->K[0] * o.c_alpha;
  a.KC1 = p->K[1] * o.c_alpha;
  a.KC2 = p->K[2] * o.c_alpha;
  a.max_u = (int)tp.max_u;
  if (cg) a.cg = *cg;
  if (tp.n_aitems > 0 && diag) {
    // two LDS rows per wavefront: four wavefronts up to 2560 nodes, else two
    const int nw = tp.max_u <= 2560 ? 4 : 2;
    k_tube_diag<<<(unsigned)tp.n_aitems, 64 * nw, sizeof(double) * 2 * nw * tp.max_u, s>>>(a);
  } else if (tp.n_aitems > 0) {
    // x and a part per wavefront: 160 KB at the 4096 nodes a tube may have
    k_tube_apply<<<(unsigned)tp.n_aitems, 64 * kApplyWaves, sizeof(double) * (1 + kApplyWaves) * tp.max_u, s>>>(a);
  }
  k_tube_sum<<<op_blocks(m->ndof, cg != nullptr), 256, 0, s>>>(tp.row_off, tp.row_ts, tp.u_off, tp.seg_off, tp.part,
                                                                m->ndof, y, x, a.cg);
  FPDE_HIP(hipGetLastError());
  return FPDE_OK;
}

// Bound by the entry loads and the same-node lanes of the LDS updates.  Per
// product 0.12 ms for 19 672 elements (11 points; 0.97 ms with the dots and the
// gather over the transpose, its values put in order once), 0.11 ms for 42 077
// elements (4 points; 0.37 ms in order already), 1.6 ms for 151 907 elements
// (11 points; 3.9 ms on merged entries, whose order cost 8 ms per assembly).
int apply_matfree(fpde_mesh *m, Plan *P, const fpde_params *p, const double *x, double *y, hipStream_t s,
                  const CgStep *cg) {
  if (m->ndof == 0) return FPDE_OK;
  const long t = timer_begin(m, s, FPDE_STAGE_APPLY);
  FPDE_TRY(apply_tubes(m, *P, p, x, y, false, s, cg));
  timer_end(m, FPDE_STAGE_APPLY, t, s);
  return FPDE_OK;
}

int matfree_diagonal(fpde_mesh *m, Plan *P, const fpde_params *p, double *d, hipStream_t s) {
  return apply_tubes(m, *P, p, nullptr, d, true, s, nullptr);
}

int launch_contract_tubes(fpde_mesh *m, Plan &P, const fpde_params *p, void *A, int64_t lda, hipStream_t s) {
  if (m->ndof == 0) return FPDE_OK;
  const long t = timer_begin(m, s, FPDE_STAGE_CONTRACT);
  FPDE_TRY(accumulate_tube_blocks(m, P, p, s));
  GatherArgs gch;
  FPDE_TRY(gather_args(m, P, lda, s, gch));
  const unsigned grid = gather_grid(m->ndof);
  // deterministic: one wavefront per row takes the row's tube slices in order
  const unsigned gthreads = p->deterministic ? 64 : 256;
  if (p->precision == FPDE_MIXED)
    k_tube_gather<float><<<grid, gthreads, sizeof(double) * gch.chunk, s>>>(gch, (float *)A);
  else
    k_tube_gather<double><<<grid, gthreads, sizeof(double) * gch.chunk, s>>>(gch, (double *)A);
  timer_end(m, FPDE_STAGE_CONTRACT, t, s);
  FPDE_HIP(hipGetLastError());
  return FPDE_OK;
}

// General form: blocks by k_tube_form from the plan's two value sets (trial
// orders in ent_val, test orders in ent_val2), with coefficients cl, cr per
// axis or, when coef is not null, per Gauss point (cl_i at [i G + g], cr_i at
// [(3 + i) G + g]), then the same row pass as the Riesz matrix.
int launch_form_tubes(fpde_mesh *m, Plan &P, const double cl[3], const double cr[3], const double *coef, double *A,
                      int64_t lda, hipStream_t s) {
  if (m->ndof == 0) return FPDE_OK;
  TubePlan &tp = P.tubes;
  if (!tp.blk) FPDE_TRY(dalloc(&tp.blk, tp.blk_n > 0 ? tp.blk_n : 1));
  AccumArgs a{};
  a.tube_off = tp.tube_off;
  a.pm = tp.pm;
  a.pw = tp.pw;
  a.items = tp.fitems;
  a.ent_slot = tp.ent_slot;
  a.ent_val = P.ent_val;
  a.val_b = P.ent_val2;
  a.blk_off = tp.blk_off;
  a.blk = tp.blk;
  a.cl0 = cl[0];
  a.cl1 = cl[1];
  a.cl2 = cl[2];
  a.cr0 = cr[0];
  a.cr1 = cr[1];
  a.cr2 = cr[2];
  a.pair = tp.pair_sorted;
  a.coef = coef;
  a.ncoef = 3 * P.G;
  if (tp.n_fitems > 0) k_tube_form<<<(unsigned)tp.n_fitems, kAccumThreads, sizeof(double) * kBand, s>>>(a);
  GatherArgs gch;
  FPDE_TRY(gather_args(m, P, lda, s, gch));
  k_tube_gather<double><<<gather_grid(m->ndof), 256, sizeof(double) * gch.chunk, s>>>(gch, A);
  FPDE_HIP(hipGetLastError());
  return FPDE_OK;
}

int launch_contract_tubes_csr(fpde_mesh *m, Plan &P, const fpde_params *p, const int64_t *row_ptr,
                              const int32_t *col, double *val, hipStream_t s) {
  if (m->ndof == 0) return FPDE_OK;
  const long t = timer_begin(m, s, FPDE_STAGE_CONTRACT);
  FPDE_TRY(accumulate_tube_blocks(m, P, p, s));
  GatherArgs gch;
  FPDE_TRY(gather_args(m, P, 0, s, gch));
  k_tube_gather_csr<<<gather_grid(m->ndof), p->deterministic ? 64 : 256, sizeof(double) * gch.chunk, s>>>(
      gch, row_ptr, col, val);
  timer_end(m, FPDE_STAGE_CONTRACT, t, s);
  FPDE_HIP(hipGetLastError());
  return FPDE_OK;
}

}  // namespace fpde
