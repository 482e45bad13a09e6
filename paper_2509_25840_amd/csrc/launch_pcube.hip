// Launches of k_pcube and k_pcube_s.
#include "launch.h"

namespace chfpe {

template <typename K, typename T, typename TO>
void launch_pcube_k(chfpe_ctx *c, K kern, size_t lds, const Batch &b, const T *X, TO *out, const double *grad) {
  allow_lds(kern, lds);
  hipLaunchKernelGGL(kern, dim3(b.pcb.nblk), dim3(c->ln.pcube_threads), lds, c->stream, b.g, c->tb, b.pcb,
                     X, out, grad);
}

// k_pcube, or its streamed form k_pcube_s where the plan chose it (p_1 axes
// up to 32 points, plain stencils; closure tables take k_pcube)
template <typename T, typename TO, int NB1, bool SPLIT, bool PERTURB>
void launch_pcube_s(chfpe_ctx *c, const Batch &b, const T *X, TO *out, const double *grad) {
  const int pad = b.pcb.rs - b.pcb.N3;
  if constexpr (kClosureBuilt<T, TO, NB1>) {
    if (c->closure_on) {
      launch_pcube_k(c, k_pcube<T, TO, NB1, SPLIT, PERTURB, true>, pcube_lds_bytes(c->d, sizeof(T), pad, false),
                     b, X, out, grad);
      return;
    }
  }
  if constexpr (NB1 <= 32) {
    if (c->ln.pcube_s) {
      launch_pcube_k(c, k_pcube_s<T, TO, NB1, PERTURB>, pcube_lds_bytes(c->d, sizeof(T), pad, true), b, X,
                     out, grad);
      return;
    }
  }
  launch_pcube_k(c, k_pcube<T, TO, NB1, SPLIT, PERTURB>, pcube_lds_bytes(c->d, sizeof(T), pad, false), b, X, out,
                 grad);
}

template <typename T, typename TO, int NB1, bool PERTURB>
void launch_pcube_n(chfpe_ctx *c, const Batch &b, const T *X, TO *out, const double *grad) {
  if (c->ln.pcube_split)
    launch_pcube_s<T, TO, NB1, true, PERTURB>(c, b, X, out, grad);
  else
    launch_pcube_s<T, TO, NB1, false, PERTURB>(c, b, X, out, grad);
}

template <typename T, typename TO, bool PERTURB>
void launch_pcube_t(chfpe_ctx *c, const Batch &b, const T *X, TO *out, const double *grad) {
  switch (c->ln.pcube_nb1) {
    case 8: launch_pcube_n<T, TO, 8, PERTURB>(c, b, X, out, grad); break;
    case 12: launch_pcube_n<T, TO, 12, PERTURB>(c, b, X, out, grad); break;
    case 16: launch_pcube_n<T, TO, 16, PERTURB>(c, b, X, out, grad); break;
    case 24: launch_pcube_n<T, TO, 24, PERTURB>(c, b, X, out, grad); break;
    case 32: launch_pcube_n<T, TO, 32, PERTURB>(c, b, X, out, grad); break;
    default: launch_pcube_n<T, TO, 48, PERTURB>(c, b, X, out, grad); break;
  }
}

#define CHFPE_INST(T, TO, P) template void launch_pcube_t<T, TO, P>(chfpe_ctx *, const Batch &, const T *, TO *, const double *);
CHFPE_INST(double, double, false)
CHFPE_INST(float, float, false)
CHFPE_INST(double, double, true)
CHFPE_INST(double, float, true)

}  // namespace chfpe
