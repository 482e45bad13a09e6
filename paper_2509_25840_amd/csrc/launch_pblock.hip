// Launches of k_pblock.
#include "launch.h"

namespace chfpe {

template <typename T, typename TO, int NMAX, int RPT, int MM, bool PERTURB>
void launch_pblock_rpt(chfpe_ctx *c, const Batch &b, const T *X, TO *out, const double *grad) {
  const Launch &ln = c->ln;
  if constexpr (kClosureBuilt<T, TO, NMAX>) {
    if (c->closure_on) {
      auto kern = k_pblock<T, TO, NMAX, RPT, MM, PERTURB, true>;
      allow_lds(kern, ln.pb_lds);
      hipLaunchKernelGGL(kern, dim3(b.pb.nblk), dim3(ln.pb_threads), ln.pb_lds, c->stream, b.g, c->tb, b.pb,
                         X, out, grad);
      return;
    }
  }
  auto kern = k_pblock<T, TO, NMAX, RPT, MM, PERTURB>;
  allow_lds(kern, ln.pb_lds);
  hipLaunchKernelGGL(kern, dim3(b.pb.nblk), dim3(ln.pb_threads), ln.pb_lds, c->stream, b.g, c->tb, b.pb, X,
                     out, grad);
}

template <typename T, typename TO, int NMAX, int MM, bool PERTURB>
void launch_pblock_nm(chfpe_ctx *c, const Batch &b, const T *X, TO *out, const double *grad) {
  if constexpr (NMAX == 24 && MM >= 2) {
    if (c->ln.pb_rpt == 3) {
      launch_pblock_rpt<T, TO, NMAX, 3, MM, PERTURB>(c, b, X, out, grad);
      return;
    }
  }
  launch_pblock_rpt<T, TO, NMAX, kPBlockRPT, MM, PERTURB>(c, b, X, out, grad);
}

template <typename T, typename TO, int NMAX, bool PERTURB>
void launch_pblock_n(chfpe_ctx *c, const Batch &b, const T *X, TO *out, const double *grad) {
  switch (c->d.M) {
    case 1: launch_pblock_nm<T, TO, NMAX, 1, PERTURB>(c, b, X, out, grad); break;
    case 2: launch_pblock_nm<T, TO, NMAX, 2, PERTURB>(c, b, X, out, grad); break;
    default: launch_pblock_nm<T, TO, NMAX, 3, PERTURB>(c, b, X, out, grad); break;
  }
}

template <typename T, typename TO, bool PERTURB>
void launch_pblock_t(chfpe_ctx *c, const Batch &b, const T *X, TO *out, const double *grad) {
  switch (c->ln.pb_nmax) {
    case 8: launch_pblock_n<T, TO, 8, PERTURB>(c, b, X, out, grad); break;
    case 12: launch_pblock_n<T, TO, 12, PERTURB>(c, b, X, out, grad); break;
    case 16: launch_pblock_n<T, TO, 16, PERTURB>(c, b, X, out, grad); break;
    case 24: launch_pblock_n<T, TO, 24, PERTURB>(c, b, X, out, grad); break;
    case 32: launch_pblock_n<T, TO, 32, PERTURB>(c, b, X, out, grad); break;
    default: launch_pblock_n<T, TO, 48, PERTURB>(c, b, X, out, grad); break;
  }
}

#define CHFPE_INST(T, TO, P) template void launch_pblock_t<T, TO, P>(chfpe_ctx *, const Batch &, const T *, TO *, const double *);
CHFPE_INST(double, double, false)
CHFPE_INST(float, float, false)
CHFPE_INST(double, double, true)
CHFPE_INST(double, float, true)

}  // namespace chfpe
