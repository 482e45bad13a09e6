// Launches of k_one.
#include "launch.h"

namespace chfpe {

// RK4 steps of one launch: a few milliseconds, so that no launch of a long
// propagation holds its compute unit for seconds.
constexpr long long kOneSteps = 256;

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
  const int nmax = std::max(a.Nq, a.Np);
  auto go = [&](bool f, long long n, long long steps, double *out) {
    a.first = f;
    a.n_samples = (int)n;
    a.stride = (int)steps;
    if (nmax <= 16)
      launch_one_ne<T, 16>(c, nb, a, states, out);
    else if (nmax <= 32)
      launch_one_ne<T, 32>(c, nb, a, states, out);
    else
      launch_one_ne<T, 48>(c, nb, a, states, out);
  };
  for (long long j = 0; j < n_samples;) {
    long long left = j == 0 && first ? 0 : stride;
    for (; left > kOneSteps; left -= kOneSteps) go(false, 1, kOneSteps, nullptr);
    // further samples with this one, as far as the step limit allows
    const long long more = stride > kOneSteps ? 0 : std::min(n_samples - j - 1, (kOneSteps - left) / std::max(1LL, stride));
    if (more > 0)
      go(left == 0, more + 1, stride, R ? R + j * ostride : nullptr);
    else
      go(left == 0, 1, left, R ? R + j * ostride : nullptr);
    j += 1 + more;
  }
}

template void launch_one<double>(chfpe_ctx *, int, double *, long long, long long, bool, double, double *, long long, int);
template void launch_one<float>(chfpe_ctx *, int, float *, long long, long long, bool, double, double *, long long, int);

}  // namespace chfpe
