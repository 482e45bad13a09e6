// Launches of k_hcube and k_hwave (Hermite basis).
#include "launch.h"

namespace chfpe {

// Hermite basis: one k_hcube launch computes the right-hand side of X and
// the stage update (EPI, coefficient cst) over every (branch, element, k).
template <typename T, int NB1, int EPI>
void launch_hcube_n(chfpe_ctx *c, const Batch &b, const T *X, const T *y, T *xo, double cst) {
  const size_t lds = (kHCubeCF + 2 * (size_t)kHCubePL * b.hcb.N2 * b.hcb.rs) * sizeof(T);
  auto kern = k_hcube<T, NB1, EPI>;
  allow_lds(kern, lds);
  hipLaunchKernelGGL(kern, dim3(b.hcb.nblk), dim3(c->ln.hcube_threads), lds, c->stream, b.g, c->tb, b.hcb, X, y,
                     xo, cst);
}

template <typename T, int EPI>
void launch_hcube(chfpe_ctx *c, const Batch &b, const T *X, const T *y, T *xo, double cst) {
  switch (c->ln.hcube_nb1) {
    case 8: launch_hcube_n<T, 8, EPI>(c, b, X, y, xo, cst); break;
    case 12: launch_hcube_n<T, 12, EPI>(c, b, X, y, xo, cst); break;
    case 16: launch_hcube_n<T, 16, EPI>(c, b, X, y, xo, cst); break;
    case 24: launch_hcube_n<T, 24, EPI>(c, b, X, y, xo, cst); break;
    case 32: launch_hcube_n<T, 32, EPI>(c, b, X, y, xo, cst); break;
    default: launch_hcube_n<T, 48, EPI>(c, b, X, y, xo, cst); break;
  }
}

// The wave-plane form of the same launch.
template <typename T, int NB, int NVR, int MM>
void launch_hwave_k(chfpe_ctx *c, const Batch &b, const T *X, const T *y, T *xo, double cst, int epi) {
  const int nw = hwave_nw(c->d, b.hcb, NB);
  const size_t lds = sizeof(T) * hwave_lds_vals(NB, b.hcb.N1, b.hcb.N2, b.hcb.N3, nw, hwave_ps(NB, NVR == 0, MM), MM);
  PCube p = b.hcb;
  if (MM == 2) {  // workgroups of nw tasks
    p.chunk = p.chunk > 0 ? std::max(1, p.chunk / nw) : 0;
    p.nblk = hcube_nblk((p.ntasks + nw - 1) / nw, p.chunk);
  }
  auto kern = k_hwave<T, NB, NVR, MM>;
  allow_lds(kern, lds);
  hipLaunchKernelGGL(kern, dim3(p.nblk), dim3(64 * nw), lds, c->stream, b.g, c->tb, p, X, y, xo, cst, epi);
}

template <typename T, int NB, int MM>
void launch_hwave_n(chfpe_ctx *c, const Batch &b, const T *X, const T *y, T *xo, double cst, int epi) {
  constexpr int full = wave_nv(NB, 1, 1);
  const PCube &p = b.hcb;
  if ((MM == 2 || p.N1 == NB) && p.N2 == NB && p.N3 == NB)
    return launch_hwave_k<T, NB, 0, MM>(c, b, X, y, xo, cst, epi);
  if constexpr (NB >= 24)
    if (p.plane <= 64 * 6) return launch_hwave_k<T, NB, 6, MM>(c, b, X, y, xo, cst, epi);
  launch_hwave_k<T, NB, full, MM>(c, b, X, y, xo, cst, epi);
}

template <typename T>
void launch_hwave(chfpe_ctx *c, const Batch &b, const T *X, const T *y, T *xo, double cst, int epi) {
#define CHFPE_HW(N) (c->d.M == 2 ? launch_hwave_n<T, N, 2>(c, b, X, y, xo, cst, epi) : launch_hwave_n<T, N, 3>(c, b, X, y, xo, cst, epi))
  switch (c->ln.hwave_nb) {
    case 8: CHFPE_HW(8); break;
    case 12: CHFPE_HW(12); break;
    case 16: CHFPE_HW(16); break;
    case 24: CHFPE_HW(24); break;
    default: launch_hwave_n<T, 32, 2>(c, b, X, y, xo, cst, epi); break;
  }
#undef CHFPE_HW
}

#define CHFPE_INST(T, EPI) \
  template void launch_hcube<T, EPI>(chfpe_ctx *, const Batch &, const T *, const T *, T *, double);
#define CHFPE_INST_T(T)    \
  CHFPE_INST(T, EPI_H1)    \
  CHFPE_INST(T, EPI_H2)    \
  CHFPE_INST(T, EPI_H4)    \
  template void launch_hwave<T>(chfpe_ctx *, const Batch &, const T *, const T *, T *, double, int);
CHFPE_INST(double, EPI_OUT)
CHFPE_INST_T(double)
CHFPE_INST_T(float)

}  // namespace chfpe
