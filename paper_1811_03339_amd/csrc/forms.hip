// The general uniform form of Sec. 1 (eq. equ:varsss), the test operator
// on the side opposite to the trial one, with the element quadrature of
// Sec. 2.1:
//
//   K_kl = sum_i sum_g w_g [cl_i(x_g) D_L^{a_i} psi_l(x_g) D_R^{b_i} psi_k(x_g)
//                         + cr_i(x_g) D_R^{a_i} psi_l(x_g) D_L^{b_i} psi_k(x_g)],
//
// trial orders a_i and test orders b_i in [0, 1] (order 0 is the identity,
// order 1 the classical derivative, D_R^1 = -d/dx), row k = test function.
// The Riesz split (a = b, cl = cr = K_i c_alpha) and the problem of Sec. 3
// (b = 1, cl = p_i, cr = q_i) are instances.
//
// Every half-ray's values are computed twice from the plan's segments: at the
// trial orders into the plan's first value set and at the test orders into its
// second.  The products are then accumulated by tubes (the two products of every
// pair into a tube block, weighted by the pair's coefficients, then the row pass
// of the Riesz matrix).  Coefficients per Gauss point went through a gather over
// each node's incidences before: 2.3 ms against 0.24 ms for 1 133 unknowns (11
// points), 89 against 14 ms for 3 x 3 x 400 cells (4 points).
#include <cmath>

#include "fpde_internal.h"

namespace fpde {

namespace {

int check_form(const fpde_mesh *m, const fpde_form_params *p) {
  if (!m || !p) return FPDE_EINVAL;
  for (int i = 0; i < 3; i++) {
    if (!(p->alpha[i] >= 0.0 && p->alpha[i] <= 1.0)) return FPDE_EALPHA;
    if (!(p->beta[i] >= 0.0 && p->beta[i] <= 1.0)) return FPDE_EALPHA;
    if (!std::isfinite(p->cl[i]) || !std::isfinite(p->cr[i])) return FPDE_EINVAL;
  }
  if (p->quad_points != 4 && p->quad_points != 11) return FPDE_EINVAL;
  if (p->coef != FPDE_COEF_CONST && p->coef != FPDE_COEF_USER) return FPDE_EINVAL;
  return FPDE_OK;
}

}  // namespace

}  // namespace fpde

using namespace fpde;

extern "C" int fpde_form_assemble(fpde_mesh *m, const fpde_form_params *p, const double *coef, double *A,
                                  int64_t lda, void *stream) {
  FPDE_TRY(check_form(m, p));
  if (!A || lda < m->ndof) return FPDE_EINVAL;
  if (p->coef == FPDE_COEF_USER && !coef) return FPDE_EINVAL;
  if (m->ndof == 0) return FPDE_OK;
  hipStream_t s = S(stream);
  Plan *P = nullptr;
  FPDE_TRY(plan_for(m, p->quad_points, p->max_steps, s, &P));
  FPDE_TRY(ensure_values_axes(m, P, p->alpha, s, 0));
  FPDE_TRY(ensure_values_axes(m, P, p->beta, s, 1));
  const long t = timer_begin(m, s, FPDE_STAGE_FORM);
  FPDE_TRY(launch_form_tubes(m, *P, p->cl, p->cr, p->coef == FPDE_COEF_USER ? coef : nullptr, A, lda, s));
  timer_end(m, FPDE_STAGE_FORM, t, s);
  FPDE_HIP(hipGetLastError());
  const int f = take_flag(m, s);
  if (f != 0) {
    invalidate_values(P);
    return f < 0 ? f : FPDE_EHIP;
  }
  return FPDE_OK;
}
