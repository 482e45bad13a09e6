// Launches of k_qpass for one arithmetic type (launch_qpass_f64.hip, _f32.hip).
#pragma once

#include "launch.h"

namespace chfpe {

template <typename T, typename TO, int NMAX, bool TWO, int EPI, int FA, int FB>
void launch_q_n(chfpe_ctx *c, const Batch &b, const QPass &qp, int threads, size_t lds, const T *X, TO *Tacc,
                const TO *y, TO *xo, const double *grad, double cst) {
  if constexpr (kClosureBuilt<T, TO, NMAX>) {
    if (c->closure_on) {
      auto kern = k_qpass<T, TO, NMAX, TWO, EPI, FA, FB, true>;
      allow_lds(kern, lds);
      hipLaunchKernelGGL(kern, dim3(qp.nblk), dim3(threads), lds, c->stream, b.g, c->tb, qp, X, Tacc, y, xo,
                         grad, cst);
      return;
    }
  }
  auto kern = k_qpass<T, TO, NMAX, TWO, EPI, FA, FB>;
  allow_lds(kern, lds);
  hipLaunchKernelGGL(kern, dim3(qp.nblk), dim3(threads), lds, c->stream, b.g, c->tb, qp, X, Tacc, y, xo, grad,
                     cst);
}

template <typename T, typename TO, bool TWO, int EPI, int FA, int FB>
void launch_q_t(chfpe_ctx *c, const Batch &b, const QPass &qp, int threads, size_t lds, int nmax, const T *X,
                TO *Tacc, const TO *y, TO *xo, const double *grad, double cst) {
  lds = lds / sizeof(double) * sizeof(T);  // the plan's tile is one of doubles
#define CHFPE_QN(N) launch_q_n<T, TO, N, TWO, EPI, FA, FB>(c, b, qp, threads, lds, X, Tacc, y, xo, grad, cst)
  switch (nmax) {
    case 8: CHFPE_QN(8); break;
    case 12: CHFPE_QN(12); break;
    case 16: CHFPE_QN(16); break;
    case 24: CHFPE_QN(24); break;
    case 32: CHFPE_QN(32); break;
    default: CHFPE_QN(48); break;
  }
#undef CHFPE_QN
}

#define CHFPE_INST(T, TO, TWO, EPI, FA, FB)                                                                        \
  template void launch_q_t<T, TO, TWO, EPI, FA, FB>(chfpe_ctx *, const Batch &, const QPass &, int, size_t, int, \
                                                    const T *, TO *, const TO *, TO *, const double *, double);
#define CHFPE_INST_STAGE(T, EPI)               \
  CHFPE_INST(T, T, false, EPI, FQ, FQ)         \
  CHFPE_INST(T, T, true, EPI, FQ, FQ)          \
  CHFPE_INST(T, T, true, EPI, FQ, FP)

}  // namespace chfpe
