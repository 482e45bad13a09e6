// Launchers of the kernel families, one translation unit each.
#pragma once

#include "context.h"

namespace chfpe {

// p side of a right-hand side (PERTURB: of X^x, dX/dq_s in grad): out from X.
template <typename T, typename TO, bool PERTURB>
void launch_pblock_t(chfpe_ctx *c, const Batch &b, const T *X, TO *out, const double *grad);
template <typename T, typename TO, bool PERTURB>
void launch_pcube_t(chfpe_ctx *c, const Batch &b, const T *X, TO *out, const double *grad);
template <typename T, typename TO, bool PERTURB>
void launch_pwave(chfpe_ctx *c, const Batch &b, const T *X, TO *out, const double *grad);
template <typename T, typename TO, bool PERTURB>
void launch_pwave2(chfpe_ctx *c, const Batch &b, const T *X, TO *out, const double *grad);
// k_qpass over the axes of qp.
template <typename T, typename TO, bool TWO, int EPI, int FA, int FB>
void launch_q_t(chfpe_ctx *c, const Batch &b, const QPass &qp, int threads, size_t lds, int nmax, const T *X,
                TO *Tacc, const TO *y, TO *xo, const double *grad, double cst);
// k_qcube: every q derivative of X added to Tacc, and the stage update epi.
template <typename T>
void launch_qcube(chfpe_ctx *c, const Batch &b, const T *X, const T *Tacc, const T *y, T *xo, double cst, int epi);
// Hermite basis: the right-hand side of X and the stage update (EPI,
// coefficient cst) over every (branch, element, k).
template <typename T, int EPI>
void launch_hcube(chfpe_ctx *c, const Batch &b, const T *X, const T *y, T *xo, double cst);
template <typename T>
void launch_hwave(chfpe_ctx *c, const Batch &b, const T *X, const T *y, T *xo, double cst, int epi);
// k_one: nb states propagated by n_samples times `stride` RK4 steps (none
// before the first sample if `first`); R (may be null) receives <C> of state b
// after sample j at j * ostride + b * bstride.
template <typename T>
void launch_one(chfpe_ctx *c, int nb, T *states, long long n_samples, long long stride, bool first, double dt, double *R,
                long long ostride, int bstride);

}  // namespace chfpe
