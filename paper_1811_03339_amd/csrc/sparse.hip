// Sparse storage of the fractional stiffness matrix on the template of
// Sec. 2.3 (Table 1), and a Krylov solve that needs no dense matrix.
//
// The template T (node j, node k) is set when, for some axis i, the boxes of
// the two element patches overlap in both coordinates other than i; it
// contains the nonzero pattern of K and its density falls like 1/N^(2/3) as
// the mesh is refined, so at large N K is kept as a CSR matrix on T instead
// of densely:
//   k_tpl_count / k_tpl_fill  one workgroup per row: every node's box tested
//                             against the row's (the patch boxes are the
//                             template's), counted, then written in column
//                             order (ballot + prefix within the workgroup);
//   assembly                  the tube accumulation, its row pass keeping the
//                             template's columns only (tubes.hip);
//   k_csr_apply               y = K x, one wavefront per row;
//   CG                        Jacobi-preconditioned conjugate gradients on
//                             either the CSR matrix or the matrix-free
//                             product of the derivative vectors (no N^2
//                             storage at all); the diagonal of K comes from
//                             the CSR row or, matrix-free, from the pairs of
//                             half-rays that both meet a node.
#include <algorithm>
#include <cmath>
#include <vector>

#include "cg.h"
#include "fpde_internal.h"

namespace fpde {

namespace {

__device__ __forceinline__ bool boxes_meet2(const double *a, const double *b) {
  bool ov[3];
#pragma unroll
  for (int d = 0; d < 3; d++) ov[d] = a[d] <= b[3 + d] && b[d] <= a[3 + d];
  return (ov[1] && ov[2]) || (ov[2] && ov[0]) || (ov[0] && ov[1]);
}

__global__ void __launch_bounds__(256) k_tpl_count(const double *__restrict__ box, int64_t n,
                                                   int64_t *__restrict__ cnt) {
  __shared__ int64_t red[4];
  const int64_t j = blockIdx.x;
  double bj[6];
#pragma unroll
  for (int d = 0; d < 6; d++) bj[d] = box[6 * j + d];
  int64_t c = 0;
  for (int64_t k = threadIdx.x; k < n; k += blockDim.x) {
    double bk[6];
#pragma unroll
    for (int d = 0; d < 6; d++) bk[d] = box[6 * k + d];
    c += boxes_meet2(bj, bk) ? 1 : 0;
  }
  for (int o = 32; o > 0; o >>= 1) c += __shfl_down(c, o, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) cnt[j] = (red[0] + red[1]) + (red[2] + red[3]);
}

// columns of row j in increasing order: 256 candidates per round, each
// thread's position = set flags before it (wave ballots + wave totals)
__global__ void __launch_bounds__(256) k_tpl_fill(const double *__restrict__ box, int64_t n,
                                                  const int64_t *__restrict__ row_ptr,
                                                  int32_t *__restrict__ col) {
  __shared__ int wtot[4];
  const int64_t j = blockIdx.x;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  double bj[6];
#pragma unroll
  for (int d = 0; d < 6; d++) bj[d] = box[6 * j + d];
  int64_t base = row_ptr[j];
  for (int64_t k0 = 0; k0 < n; k0 += blockDim.x) {
    const int64_t k = k0 + threadIdx.x;
    bool hit = false;
    if (k < n) {
      double bk[6];
#pragma unroll
      for (int d = 0; d < 6; d++) bk[d] = box[6 * k + d];
      hit = boxes_meet2(bj, bk);
    }
    const unsigned long long bal = __ballot(hit);
    const int before = __popcll(bal & ((1ull << lane) - 1ull));
    if (lane == 0) wtot[w] = __popcll(bal);
    __syncthreads();
    int off = 0;
    for (int v = 0; v < w; v++) off += wtot[v];
    const int tot = (wtot[0] + wtot[1]) + (wtot[2] + wtot[3]);
    if (hit) col[base + off + before] = (int32_t)k;
    base += tot;
    __syncthreads();  // wtot is rewritten next round
  }
}

// y = K x, one wavefront per row (4 rows per workgroup and step); c as in CgStep
__global__ void __launch_bounds__(256) k_csr_apply(const int64_t *__restrict__ row_ptr,
                                                   const int32_t *__restrict__ col, const double *__restrict__ val,
                                                   const double *__restrict__ x, int64_t n, double *__restrict__ y,
                                                   CgStep c) {
  __shared__ double red[4];
  double be = 0.0;
  if (c.st && cg_ended(c, be, red, blockIdx.x == 0)) return;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  double xy = 0.0;
  for (int64_t j = (int64_t)blockIdx.x * 4 + w; j < n; j += (int64_t)gridDim.x * 4) {
    double s = 0.0;
    for (int64_t q = row_ptr[j] + lane; q < row_ptr[j + 1]; q += 64) s = fma(val[q], cg_entry(c, be, x, col[q]), s);
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
  __syncthreads();  // red
  if (lane == 0) red[w] = xy;
  __syncthreads();
  if (threadIdx.x == 0) c.dot[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

// d_j = K_jj from the CSR row (binary search of the sorted columns)
__global__ void k_csr_diag(const int64_t *__restrict__ row_ptr, const int32_t *__restrict__ col,
                           const double *__restrict__ val, int64_t n, double *__restrict__ d) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n) return;
  int64_t lo = row_ptr[j], hi = row_ptr[j + 1];
  double v = 0.0;
  while (lo < hi) {
    const int64_t mid = lo + (hi - lo) / 2;
    const int32_t c = col[mid];
    if (c == (int32_t)j) {
      v = val[mid];
      break;
    }
    if (c < (int32_t)j) lo = mid + 1;
    else hi = mid;
  }
  d[j] = v;
}

// ---- Conjugate gradients without host round trips ----
//
// The scalars of the iteration stay on the device: a kernel leaves partial
// sums, one per workgroup, and every workgroup of the next kernel adds them up
// itself, in the same order, so that all agree without a launch in between.
// An iteration is two launches (direction and product with p.q; update with r.r
// and r.z; matrix-free one more, the row pass).  The host queues iterations a few at a time and looks at the
// state of the chunk before; what is queued past the end finds it in the state and
// does nothing.  (With three dot products per iteration read back by the host
// an iteration took 200 us around a product of 12 us, with a launch of its own
// for the direction 21 us; now 20 us.)
constexpr int kCgParts = 256;  // workgroups of the vector kernels at most

// two sums over the workgroup's threads to part[2 blockIdx.x], [.. + 1]
__device__ __forceinline__ void put_parts(double a, double b, double *__restrict__ part, double *red) {
  for (int o = 32; o > 0; o >>= 1) {
    a += __shfl_xor(a, o, 64);
    b += __shfl_xor(b, o, 64);
  }
  __syncthreads();
  if ((threadIdx.x & 63) == 0) {
    red[threadIdx.x >> 6] = a;
    red[4 + (threadIdx.x >> 6)] = b;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
    part[2 * blockIdx.x + 1] = (red[4] + red[5]) + (red[6] + red[7]);
  }
}

__global__ void k_cg_clear(CgState *st) {
  st->end = INT64_MAX;
  st->done = 0;
  st->it = 0;
}

// start: r = b, z = p = r / d, u = 0, parts of b.b and r.z
__global__ void __launch_bounds__(256) k_cg_start(const double *__restrict__ b, const double *__restrict__ d,
                                                  double *__restrict__ u, double *__restrict__ r,
                                                  double *__restrict__ z, double *__restrict__ p,
                                                  double *__restrict__ dinv, int64_t n, CgState *st,
                                                  double *__restrict__ part) {
  __shared__ double red[8];
  double bb = 0.0, rz = 0.0;
  for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < n; k += (int64_t)gridDim.x * 256) {
    const double dk = d[k], bk = b[k];
    if (!(dk > 0.0)) atomicMax(&st->done, 2);  // a diagonal entry <= 0: K is not SPD
    const double di = dk > 0.0 ? 1.0 / dk : 1.0, zk = bk * di;
    dinv[k] = di;
    u[k] = 0.0;
    r[k] = bk;
    z[k] = zk;
    p[k] = zk;
    bb = fma(bk, bk, bb);
    rz = fma(bk, zk, rz);
  }
  put_parts(bb, rz, part, red);
}

// one workgroup: the start's sums; nothing to do for b = 0 or tol >= 1
__global__ void __launch_bounds__(256) k_cg_begin(CgState *st, double tol, const double *__restrict__ part, int np) {
  __shared__ double red[4];
  const double bb = sum_parts(part, np, 2, red), rz = sum_parts(part + 1, np, 2, red);
  if (threadIdx.x == 0) {
    st->bn2 = bb;
    st->rz[0] = rz;
    st->rr = bb;
    if (st->done == 0 && !(bb > 0.0 && 1.0 > tol)) st->done = 1;
    if (st->done) st->end = -1;
  }
}

// al = r.z / p.q; u += al p; r -= al q; z = r / d; parts of r.r and r.z
__global__ void __launch_bounds__(256) k_cg_update(double *__restrict__ u, double *__restrict__ r,
                                                   double *__restrict__ z, const double *__restrict__ p,
                                                   const double *__restrict__ q, const double *__restrict__ dinv,
                                                   int64_t n, CgState *st, int it, const double *__restrict__ pq_part,
                                                   int npq, double *__restrict__ part) {
  __shared__ double red[8];
  const int64_t launch = 2 * (int64_t)it + 1;
  if (cg_over(st, launch)) return;
  const double pq = sum_parts(pq_part, npq, 1, red);
  if (!(pq > 0.0)) {  // the same in every workgroup
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      st->done = 2;
      st->end = launch;
    }
    return;
  }
  const double al = st->rz[it & 1] / pq;
  double rr = 0.0, rz = 0.0;
  for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < n; k += (int64_t)gridDim.x * 256) {
    u[k] = fma(al, p[k], u[k]);
    const double rk = fma(-al, q[k], r[k]), zk = rk * dinv[k];
    r[k] = rk;
    z[k] = zk;
    rr = fma(rk, rk, rr);
    rz = fma(rk, zk, rz);
  }
  put_parts(rr, rz, part, red);
}

// one workgroup: the end of the last iteration that may be taken
__global__ void __launch_bounds__(256) k_cg_last(CgStep c) {
  __shared__ double red[4];
  double be;
  (void)cg_ended(c, be, red, true);
}

// parts of |b - q|^2, and their sum to st->rt (one workgroup)
__global__ void __launch_bounds__(256) k_cg_residual(const double *__restrict__ b, const double *__restrict__ q,
                                                     int64_t n, double *__restrict__ part) {
  __shared__ double red[8];
  double s = 0.0;
  for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < n; k += (int64_t)gridDim.x * 256) {
    const double v = b[k] - q[k];
    s = fma(v, v, s);
  }
  put_parts(s, 0.0, part, red);
}
__global__ void __launch_bounds__(256) k_cg_end(CgState *st, const double *__restrict__ part, int np) {
  __shared__ double red[4];
  const double rt = sum_parts(part, np, 2, red);
  if (threadIdx.x == 0) st->rt = rt;
}

inline unsigned blocks_of(int64_t n, int b = 256) { return (unsigned)((n + b - 1) / b); }

// CG scratch in the mesh handle: r, z, two p, q, d, dinv (7 N), partial sums of
// the product and of the vector kernels, the state
struct CgWork {
  double *r, *z, *p[2], *q, *d, *dinv, *op_part, *part;
  CgState *st, *host;  // host: two pinned copies
};

}  // namespace

static int ensure_cg(fpde_mesh *m, CgWork *w) {
  const int64_t n = m->ndof > 0 ? m->ndof : 1;
  const int64_t need = 7 * n + kOpParts + 2 * kCgParts + (int64_t)(sizeof(CgState) / sizeof(double));
  static_assert(sizeof(CgState) % sizeof(double) == 0, "the state follows the sums");
  if (m->cg_n < need) {
    dfree(m->cg);
    m->cg_n = 0;
    FPDE_TRY(dalloc(&m->cg, (size_t)need));
    m->cg_n = need;
  }
  if (!m->hcg && hipHostMalloc(&m->hcg, 2 * sizeof(CgState), hipHostMallocDefault) != hipSuccess) {
    m->hcg = nullptr;
    return FPDE_ENOMEM;
  }
  for (hipEvent_t &e : m->cev)
    if (!e && hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess) {
      e = nullptr;
      return FPDE_EHIP;
    }
  w->r = m->cg;
  w->z = w->r + n;
  w->p[0] = w->z + n;
  w->p[1] = w->p[0] + n;
  w->q = w->p[1] + n;
  w->d = w->q + n;
  w->dinv = w->d + n;
  w->op_part = w->dinv + n;
  w->part = w->op_part + kOpParts;
  w->st = (CgState *)(w->part + 2 * kCgParts);
  w->host = (CgState *)m->hcg;
  return FPDE_OK;
}

}  // namespace fpde

using namespace fpde;

extern "C" int fpde_template_csr(fpde_mesh *m, int64_t *row_ptr, int32_t *col, int64_t capacity, int64_t *nnz,
                                 void *stream) {
  if (!m || !row_ptr || !nnz) return FPDE_EINVAL;
  hipStream_t s = S(stream);
  const int64_t n = m->ndof;
  *nnz = 0;
  if (n == 0) {
    FPDE_HIP(hipMemsetAsync(row_ptr, 0, sizeof(int64_t), s));
    FPDE_HIP(hipStreamSynchronize(s));
    return FPDE_OK;
  }
  if (n >= (int64_t(1) << 31)) return FPDE_EUNSUPPORTED;
  FPDE_TRY(ensure_patch_boxes(m, s));
  int64_t *cnt = nullptr;
  FPDE_TRY(dalloc(&cnt, (size_t)(n + 1)));
  int st = FPDE_OK;
  const long t = timer_begin(m, s, FPDE_STAGE_PLAN);
  k_tpl_count<<<(unsigned)n, 256, 0, s>>>(m->pbox, n, cnt);
  if (hipGetLastError() != hipSuccess) st = FPDE_EHIP;
  // row_ptr = exclusive prefix of the counts (host: N + 1 values)
  std::vector<int64_t> h(n + 1);
  if (st == FPDE_OK && hipMemcpyAsync(h.data(), cnt, sizeof(int64_t) * n, hipMemcpyDeviceToHost, s) != hipSuccess)
    st = FPDE_EHIP;
  if (st == FPDE_OK && hipStreamSynchronize(s) != hipSuccess) st = FPDE_EHIP;
  if (st == FPDE_OK) {
    int64_t acc = 0;
    for (int64_t j = 0; j < n; j++) {
      const int64_t c = h[j];
      h[j] = acc;
      acc += c;
    }
    h[n] = acc;
    *nnz = acc;
    if (hipMemcpyAsync(row_ptr, h.data(), sizeof(int64_t) * (n + 1), hipMemcpyHostToDevice, s) != hipSuccess)
      st = FPDE_EHIP;
  }
  if (st == FPDE_OK && col) {
    if (capacity < *nnz) {
      st = FPDE_EINVAL;
    } else {
      k_tpl_fill<<<(unsigned)n, 256, 0, s>>>(m->pbox, n, row_ptr, col);
      if (hipGetLastError() != hipSuccess) st = FPDE_EHIP;
    }
  }
  timer_end(m, FPDE_STAGE_PLAN, t, s);
  if (hipStreamSynchronize(s) != hipSuccess && st == FPDE_OK) st = FPDE_EHIP;
  dfree(cnt);
  return st;
}

extern "C" int fpde_assemble_csr(fpde_mesh *m, const fpde_params *p, const int64_t *row_ptr, const int32_t *col,
                                 double *val, double *b, const double *f_gauss, void *stream) {
  FPDE_TRY(check_params(m, p));
  if (!row_ptr || !col || !val) return FPDE_EINVAL;
  if (p->precision != FPDE_FP64) return FPDE_EUNSUPPORTED;
  if (p->source == FPDE_SRC_USER && !f_gauss && b) return FPDE_EINVAL;
  hipStream_t s = S(stream);
  Plan *P = nullptr;
  FPDE_TRY(plan_for(m, p->quad_points, p->max_steps, s, &P));
  FPDE_TRY(ensure_values(m, P, p->alpha, s));
  FPDE_TRY(launch_contract_tubes_csr(m, *P, p, row_ptr, col, val, s));
  if (b) FPDE_TRY(launch_load(m, p, b, f_gauss, s));
  const int f = take_flag(m, s);
  if (f != 0) {
    invalidate_values(P);
    return f < 0 ? f : FPDE_EHIP;
  }
  return FPDE_OK;
}

extern "C" int fpde_csr_apply(fpde_mesh *m, const int64_t *row_ptr, const int32_t *col, const double *val,
                              const double *x, double *y, void *stream) {
  if (!m || !row_ptr || !col || !val || !x || !y) return FPDE_EINVAL;
  if (m->ndof == 0) return FPDE_OK;
  hipStream_t s = S(stream);
  const long t = timer_begin(m, s, FPDE_STAGE_SPMV);
  k_csr_apply<<<op_blocks(m->ndof, false), 256, 0, s>>>(row_ptr, col, val, x, m->ndof, y, CgStep{});
  timer_end(m, FPDE_STAGE_SPMV, t, s);
  FPDE_HIP(hipGetLastError());
  return FPDE_OK;
}

extern "C" int fpde_cg_solve(fpde_mesh *m, const fpde_params *p, const int64_t *row_ptr, const int32_t *col,
                             const double *val, const double *b, double *u, double tol, int max_iter,
                             fpde_solve_info *info, void *stream) {
  FPDE_TRY(check_params(m, p));
  if (!b || !u || b == u) return FPDE_EINVAL;
  const bool csr = row_ptr != nullptr;
  if (csr && (!col || !val)) return FPDE_EINVAL;
  if (info) {
    info->ir_iters = 0;
    info->final_rel_residual = 0.0;
    info->failed_pivot = -1;
  }
  const int64_t n = m->ndof;
  if (n == 0) return FPDE_OK;
  if (!(tol > 0.0)) tol = 1e-10;
  if (max_iter <= 0) max_iter = 10000;
  hipStream_t s = S(stream);
  CgWork w;
  FPDE_TRY(ensure_cg(m, &w));
  Plan *P = nullptr;
  if (!csr) {
    FPDE_TRY(plan_for(m, p->quad_points, p->max_steps, s, &P));
    FPDE_TRY(ensure_values(m, P, p->alpha, s));
  }
  // y = K x, plain or as a step of the loop
  auto op = [&](const double *x, double *y, const CgStep &c) -> int {
    if (csr) {
      const long t = timer_begin(m, s, FPDE_STAGE_SPMV);
      k_csr_apply<<<op_blocks(n, c.st != nullptr), 256, 0, s>>>(row_ptr, col, val, x, n, y, c);
      timer_end(m, FPDE_STAGE_SPMV, t, s);
      return hipGetLastError() == hipSuccess ? FPDE_OK : FPDE_EHIP;
    }
    return apply_matfree(m, P, p, x, y, s, c.st ? &c : nullptr);
  };
  const unsigned vb = (unsigned)std::min<int64_t>(blocks_of(n), kCgParts);
  const long t_all = timer_begin(m, s, FPDE_STAGE_CG);
  // diagonal of K for the Jacobi preconditioner
  if (csr) {
    k_csr_diag<<<blocks_of(n), 256, 0, s>>>(row_ptr, col, val, n, w.d);
  } else {
    FPDE_TRY(matfree_diagonal(m, P, p, w.d, s));
  }
  k_cg_clear<<<1, 1, 0, s>>>(w.st);
  k_cg_start<<<vb, 256, 0, s>>>(b, w.d, u, w.r, w.z, w.p[0], w.dinv, n, w.st, w.part);
  k_cg_begin<<<1, 256, 0, s>>>(w.st, tol, w.part, (int)vb);
  // chunks of iterations, the next one queued before the state of the last is read
  constexpr int kChunk = 4;
  int queued = 0;
  CgStep c;
  c.st = w.st;
  c.z = w.z;
  c.part = w.part;
  c.np = (int)vb;
  c.dot = w.op_part;
  c.tol = tol;
  auto chunk = [&](int slot) -> int {
    for (int k = 0; k < kChunk && queued < max_iter; k++, queued++) {
      c.it = queued;
      c.pn = w.p[(queued + 1) & 1];
      FPDE_TRY(op(w.p[queued & 1], w.q, c));
      k_cg_update<<<vb, 256, 0, s>>>(u, w.r, w.z, c.pn, w.q, w.dinv, n, w.st, queued, w.op_part,
                                     (int)op_blocks(n, true), w.part);
    }
    if (queued == max_iter) {
      c.it = queued;
      k_cg_last<<<1, 256, 0, s>>>(c);
    }
    FPDE_HIP(hipGetLastError());
    FPDE_HIP(hipMemcpyAsync(&w.host[slot], w.st, sizeof(CgState), hipMemcpyDeviceToHost, s));
    FPDE_HIP(hipEventRecord(m->cev[slot], s));
    return FPDE_OK;
  };
  FPDE_TRY(chunk(0));
  CgState st{};
  for (int slot = 0;; slot ^= 1) {
    const bool more = queued < max_iter;
    if (more) FPDE_TRY(chunk(slot ^ 1));
    FPDE_HIP(hipEventSynchronize(m->cev[slot]));
    st = w.host[slot];
    if (st.done || !more) break;
  }
  timer_end(m, FPDE_STAGE_CG, t_all, s);
  if (st.done == 2) {  // a diagonal entry or p.Kp <= 0; nothing stays queued
    FPDE_HIP(hipStreamSynchronize(s));
    return FPDE_ENOTSPD;
  }
  // the true residual b - K u of the result, not the recursively updated one
  FPDE_TRY(op(u, w.q, CgStep{}));
  k_cg_residual<<<vb, 256, 0, s>>>(b, w.q, n, w.part);
  k_cg_end<<<1, 256, 0, s>>>(w.st, w.part, (int)vb);
  FPDE_HIP(hipGetLastError());
  FPDE_HIP(hipMemcpyAsync(&w.host[0], w.st, sizeof(CgState), hipMemcpyDeviceToHost, s));
  const int f = take_flag(m, s);  // and the copy above
  const double bn = std::sqrt(w.host[0].bn2), rt = std::sqrt(w.host[0].rt);
  const double rel = bn > 0 ? std::sqrt(w.host[0].rr) / bn : 0.0;
  if (info) {
    info->ir_iters = w.host[0].it;
    info->final_rel_residual = bn > 0 ? rt / bn : rt;
  }
  if (f != 0) return f < 0 ? f : FPDE_EHIP;
  return rel <= tol ? FPDE_OK : FPDE_ENOCONV;
}
