// Launches of k_pwave.
#include "launch.h"

namespace chfpe {

// k_pwave (three modes): a cube whose axes all have NB points (NVR = 0), or any
// block of axes of at most NB points with planes of at most 64 NVR points.
template <typename T, typename TO, int NB, int NVR, bool PERTURB>
void launch_pwave_k(chfpe_ctx *c, const Batch &b, const T *X, TO *out, const double *grad) {
  const int nw = pwave_nw(b.pcb, NB);
  const size_t lds = sizeof(T) * pwave_lds_vals(NB, b.pcb.N1, b.pcb.N2, b.pcb.N3, nw, wave_ps(NB, NVR == 0),
                                                c->closure_on);
  if constexpr (kClosureBuilt<T, TO, NB>) {
    if (c->closure_on) {
      auto kern = k_pwave<T, TO, NB, NVR, PERTURB, true>;
      allow_lds(kern, lds);
      hipLaunchKernelGGL(kern, dim3(b.pcb.nblk), dim3(64 * nw), lds, c->stream, b.g, c->tb, b.pcb, X, out, grad);
      return;
    }
  }
  auto kern = k_pwave<T, TO, NB, NVR, PERTURB>;
  allow_lds(kern, lds);
  hipLaunchKernelGGL(kern, dim3(b.pcb.nblk), dim3(64 * nw), lds, c->stream, b.g, c->tb, b.pcb, X, out, grad);
}

template <typename T, typename TO, int NB, bool PERTURB>
void launch_pwave_n(chfpe_ctx *c, const Batch &b, const T *X, TO *out, const double *grad) {
  constexpr int full = wave_nv(NB, 1, 1);  // vectors per lane of an NB x NB plane, one value each
  if (b.pcb.N1 == NB && b.pcb.N2 == NB && b.pcb.N3 == NB) {
    launch_pwave_k<T, TO, NB, 0, PERTURB>(c, b, X, out, grad);
    return;
  }
  if constexpr (NB >= 24) {
    if (b.pcb.plane <= 64 * 4) return launch_pwave_k<T, TO, NB, 4, PERTURB>(c, b, X, out, grad);
    if (b.pcb.plane <= 64 * 6) return launch_pwave_k<T, TO, NB, 6, PERTURB>(c, b, X, out, grad);
  }
  if constexpr (NB == 16) {
    if (b.pcb.plane <= 64 * 2) return launch_pwave_k<T, TO, NB, 2, PERTURB>(c, b, X, out, grad);
  }
  launch_pwave_k<T, TO, NB, full, PERTURB>(c, b, X, out, grad);
}

template <typename T, typename TO, bool PERTURB>
void launch_pwave(chfpe_ctx *c, const Batch &b, const T *X, TO *out, const double *grad) {
  switch (c->ln.pwave_nb) {
    case 8: launch_pwave_n<T, TO, 8, PERTURB>(c, b, X, out, grad); break;
    case 12: launch_pwave_n<T, TO, 12, PERTURB>(c, b, X, out, grad); break;
    case 16: launch_pwave_n<T, TO, 16, PERTURB>(c, b, X, out, grad); break;
    default: launch_pwave_n<T, TO, 24, PERTURB>(c, b, X, out, grad); break;
  }
}

// k_pwave2 (two modes): a square plane of NB points on both axes (NVR = 0), or
// any plane of at most 64 NVR points with axes of at most NB points.
template <typename T, typename TO, int NB, int NVR, bool PERTURB>
void launch_pwave2_k(chfpe_ctx *c, const Batch &b, const T *X, TO *out, const double *grad) {
  const size_t lds = sizeof(T) * pwave2_lds_vals(NB, b.pw2.N2, b.pw2.N3, c->closure_on);
  auto go = [&](auto kern) {
    allow_lds(kern, lds);
    hipLaunchKernelGGL(kern, dim3(b.pw2.nblk), dim3(64 * kPWave2Waves), lds, c->stream, b.g, c->tb, b.pw2, X, out,
                       grad);
  };
  if constexpr (kClosureBuilt<T, TO, NB>) {
    if (c->closure_on) return go(k_pwave2<T, TO, NB, NVR, PERTURB, true>);
  }
  go(k_pwave2<T, TO, NB, NVR, PERTURB>);
}

template <typename T, typename TO, int NB, bool PERTURB>
void launch_pwave2_n(chfpe_ctx *c, const Batch &b, const T *X, TO *out, const double *grad) {
  constexpr int full = wave_nv(NB, 1, 1);
  if (b.pw2.N2 == NB && b.pw2.N3 == NB) return launch_pwave2_k<T, TO, NB, 0, PERTURB>(c, b, X, out, grad);
  // planes well below NB x NB: fewer registers and no loads of empty vectors (25 x
  // 5 points, 16 FP64 states, with 10, 3 vectors a lane 524, 417 us an RK4 step;
  // 32 x 8, one state, with 10, 5 101, 94; 9 x 5 with 3, 1 66, 62)
  constexpr int part = (full * 5 + 7) / 8;
  constexpr int small = NB >= 24 ? 3 : NB == 12 ? 1 : part, mid = NB >= 32 ? 5 : small;
  if constexpr (small < part)
    if (b.pw2.plane <= 64 * small) return launch_pwave2_k<T, TO, NB, small, PERTURB>(c, b, X, out, grad);
  if constexpr (mid > small)
    if (b.pw2.plane <= 64 * mid) return launch_pwave2_k<T, TO, NB, mid, PERTURB>(c, b, X, out, grad);
  if constexpr (full >= 4)
    if (b.pw2.plane <= 64 * part) return launch_pwave2_k<T, TO, NB, part, PERTURB>(c, b, X, out, grad);
  launch_pwave2_k<T, TO, NB, full, PERTURB>(c, b, X, out, grad);
}

template <typename T, typename TO, bool PERTURB>
void launch_pwave2(chfpe_ctx *c, const Batch &b, const T *X, TO *out, const double *grad) {
  switch (c->ln.pwave2_nb) {
    case 8: launch_pwave2_n<T, TO, 8, PERTURB>(c, b, X, out, grad); break;
    case 12: launch_pwave2_n<T, TO, 12, PERTURB>(c, b, X, out, grad); break;
    case 16: launch_pwave2_n<T, TO, 16, PERTURB>(c, b, X, out, grad); break;
    case 24: launch_pwave2_n<T, TO, 24, PERTURB>(c, b, X, out, grad); break;
    default: launch_pwave2_n<T, TO, 32, PERTURB>(c, b, X, out, grad); break;
  }
}

#define CHFPE_INST(T, TO, P)                                                                                \
  template void launch_pwave<T, TO, P>(chfpe_ctx *, const Batch &, const T *, TO *, const double *);        \
  template void launch_pwave2<T, TO, P>(chfpe_ctx *, const Batch &, const T *, TO *, const double *);
CHFPE_INST(double, double, false)
CHFPE_INST(float, float, false)
CHFPE_INST(double, double, true)
CHFPE_INST(double, float, true)

}  // namespace chfpe
