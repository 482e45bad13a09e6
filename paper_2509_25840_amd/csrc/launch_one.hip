// Launches of k_one.
#include "launch.h"

namespace chfpe {

template <typename T, int NB>
void launch_one_ne(chfpe_ctx *c, int nb, const OneArgs &a, T *states, double *R) {
  const Derived &d = c->d;
  const int cols = d.Nq[0] * d.Np[0];
  const int threads = std::min(kOneThreads, (cols + 63) / 64 * 64);
  const size_t lds = one_lds_vals(d) * sizeof(T);
#define CHFPE_ONE(NE)                                                                                               \
  if constexpr (one_fits(sizeof(double), NB, NE)) {                                                                                                                \
    auto kern = k_one<T, NB, NE>;                                                                                   \
    allow_lds(kern, lds);                                                                                           \
    hipLaunchKernelGGL(kern, dim3(nb), dim3(threads), lds, c->stream, c->g, c->tb, a, states, c->Cw, c->wp, R);     \
  }
  switch (one_ne(d.ne)) {
    case 1: CHFPE_ONE(1) break;
    case 2: CHFPE_ONE(2) break;
    case 4: CHFPE_ONE(4) break;
    default: CHFPE_ONE(kOneMaxElements) break;
  }
#undef CHFPE_ONE
}

template <typename T>
void launch_one(chfpe_ctx *c, int nb, T *states, long long n_samples, long long stride, bool first, double dt, double *R,
                long long ostride, int bstride) {
  const Derived &d = c->d;
  OneArgs a{};
  a.Nq = d.Nq[0];
  a.Np = d.Np[0];
  a.dt = dt;
  a.dV = c->dV;
  a.ostride = ostride;
  a.bstride = bstride;
  a.first = first;
  a.n_samples = (int)n_samples;
  a.stride = (int)stride;
  const int nmax = std::max(a.Nq, a.Np);
  if (nmax <= 16)
    launch_one_ne<T, 16>(c, nb, a, states, R);
  else if (nmax <= 32)
    launch_one_ne<T, 32>(c, nb, a, states, R);
  else
    launch_one_ne<T, 48>(c, nb, a, states, R);
}

template void launch_one<double>(chfpe_ctx *, int, double *, long long, long long, bool, double, double *, long long, int);
template void launch_one<float>(chfpe_ctx *, int, float *, long long, long long, bool, double, double *, long long, int);

}  // namespace chfpe
