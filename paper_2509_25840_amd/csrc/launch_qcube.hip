// Launches of k_qcube.
#include "launch.h"

namespace chfpe {

template <typename T, int NB>
void launch_qcube_n(chfpe_ctx *c, const Batch &b, const T *X, const T *Tacc, const T *y, T *xo, double cst, int epi) {
  constexpr int C = qcube_c(sizeof(T));
  QCube q{};
  q.nchunk = (c->d.P + C - 1) / C;
  q.ntasks = c->d.ne * b.g.nbatch * q.nchunk;
  q.nblk = pad8(q.ntasks);
  const size_t lds = sizeof(T) * qcube_lds_vals(NB, C);
  auto kern = k_qcube<T, NB>;
  allow_lds(kern, lds);
  hipLaunchKernelGGL(kern, dim3(q.nblk), dim3(NB * NB * kQcParts), lds, c->stream, b.g, c->tb, q, X, Tacc, y, xo, cst,
                     epi);
}

template <typename T>
void launch_qcube(chfpe_ctx *c, const Batch &b, const T *X, const T *Tacc, const T *y, T *xo, double cst, int epi) {
#define CHFPE_QC(N) case N: launch_qcube_n<T, N>(c, b, X, Tacc, y, xo, cst, epi); break;
  switch (c->d.Nq[0]) {
    CHFPE_QC(5) CHFPE_QC(6) CHFPE_QC(7) CHFPE_QC(8) CHFPE_QC(9) CHFPE_QC(10)
    CHFPE_QC(11) CHFPE_QC(12) CHFPE_QC(13) CHFPE_QC(14) CHFPE_QC(15)
    default: launch_qcube_n<T, 16>(c, b, X, Tacc, y, xo, cst, epi); break;
  }
#undef CHFPE_QC
}

template void launch_qcube<double>(chfpe_ctx *, const Batch &, const double *, const double *, const double *, double *,
                                   double, int);
template void launch_qcube<float>(chfpe_ctx *, const Batch &, const float *, const float *, const float *, float *,
                                  double, int);

}  // namespace chfpe
