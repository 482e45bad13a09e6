// k_one (one mode, grid basis): whole RK4 propagations of small states by one
// workgroup per state.
//
// A one-mode state is at most a few hundred kilobytes, so a launch per pass
// (eight per RK4 step) costs far more than its work.  Per RK4 step, before and
// after: 48 x 48 points, depth 3 85 -> 23 us; bound by the 96 dependent
// steps of a line solve (depth 0: 12 us) and by the instructions of one
// compute unit.  States whose arrays do not fit one workgroup's LDS (above 32
// points, depth 4 and more) keep the launches per pass, which have more units.  Here a workgroup keeps its state in
// registers and LDS over any number of steps.  Thread t owns the columns
// (q, p) = t, t + threads, ... for every element n, so the hierarchy's
// couplings stay in its registers; only the two derivatives go through LDS:
// the h_n as [q][p] and the p fields G_n as [p][q] arrays per element, so that
// every line is a column.  Observables of element 0 are summed in the
// workgroup (FP64, fixed order).
#pragma once

#include "wave.h"

namespace chfpe {

struct OneArgs {
  int Nq, Np;
  int first;              // 1: the first sample is taken before any step
  int n_samples, stride;  // samples, RK4 steps before each
  double dt, dV;
  long long ostride;      // of a sample in R
  int bstride;            // of a state in R
};

constexpr int kOneThreads = 768;
constexpr int kOneMaxElements = 7;
// Row stride of the LDS arrays for axes of at most nb points: a constant, so
// that the values of a line are one address plus constants; odd, so that lanes
// along a row and lanes down a column read distinct banks.
constexpr int one_rs(const int nb) { return nb + 1; }
constexpr int one_bucket(const int n) { return n <= 16 ? 16 : n <= 32 ? 32 : 48; }
// Both derivative arrays of ne elements of up to nb x nb points fit the LDS.
constexpr int kOneTables = 4 * kTab + 4;
constexpr bool one_fits(const int tsize, const int nb, const int ne) {
  return ((size_t)2 * ne * nb * one_rs(nb) + kOneTables) * tsize <= 160 * 1024 - 256;
}
constexpr int one_ne(const int ne) { return ne <= 2 ? ne : ne <= 4 ? 4 : kOneMaxElements; }
constexpr int one_cpt(const int nb) { return nb <= 16 ? 1 : nb <= 32 ? 2 : 3; }

template <typename T, int NB, int NE>
__global__ void __launch_bounds__(kOneThreads)
k_one(const Geom g, const Tabs tb, const OneArgs a, T *__restrict__ states, const double *__restrict__ Cw,
      const double *__restrict__ wp, double *__restrict__ R) {
  constexpr int RS = one_rs(NB), CPT = one_cpt(NB);
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ double part[kOneThreads / 64];
  const int ne = g.ne;
  const int cols = a.Nq * a.Np;
  const int arr = max(a.Nq, a.Np) * RS;  // one element's LDS array
  T *Z = reinterpret_cast<T *>(smem_raw);  // h_n, [q][p]
  T *Y = Z + ne * arr;                     // G_n, [p][q]
  // F and V' by q, p and -p/m (times cb) by p
  T *Fq = Y + ne * arr, *Vq = Fq + kTab, *Pp = Vq + kTab, *Kp = Pp + kTab;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), nw = (int)(blockDim.x >> 6);
  T *st = states + (long long)blockIdx.x * ne * g.E;
  // element factors: G_n = F h + V' (h_{n+1} + cc h_{n-1}), times cb
  T cc[NE], tc[NE], dmp[NE];
#pragma unroll
  for (int e = 0; e < NE; ++e) {
    const int ee = min(e, ne - 1);
    cc[e] = T(tb.cc[ee * 3]);
    tc[e] = T(0.5 * tb.tc[ee * 3]);
    dmp[e] = T(tb.damp[ee]);
  }
  const T bm = T(g.bm[0]);
  if (tid < a.Nq) {
    Fq[tid] = T(tb.F[tid] * g.dp_cb[0]);
    Vq[tid] = T(tb.VpQ[tid]);
  }
  if (tid < a.Np) {
    Pp[tid] = T(tb.pg[tid]);
    Kp[tid] = T(-tb.pm[tid] * g.dq_cb[0]);
  }
  const T cbp = T(g.dp_cb[0]);
  int iq[CPT], ip[CPT];
  bool live[CPT];
  T z[CPT][NE], y[CPT][NE];  // zero past the hierarchy
#pragma unroll
  for (int c = 0; c < CPT; ++c) {
    const int col = tid + c * (int)blockDim.x;
    live[c] = col < cols;
    const int cl = live[c] ? col : 0;
    iq[c] = cl / a.Np;
    ip[c] = cl - iq[c] * a.Np;
#pragma unroll
    for (int e = 0; e < NE; ++e) z[c][e] = y[c][e] = live[c] && e < ne ? st[(long long)e * cols + col] : T(0);
  }
  const int nql = ne * a.Np, npl = ne * a.Nq;  // lines along q and along p
  const int wq = (nql + 63) / 64, wpn = (npl + 63) / 64;
  __syncthreads();

  for (int s = 0; s < a.n_samples; ++s) {
    for (int step = 0; step < (s == 0 && a.first ? 0 : a.stride); ++step) {
#pragma unroll 1
      for (int k = 0; k < 4; ++k) {
        const T cst = T(k == 0 ? 0.25 * a.dt : k == 1 ? a.dt / 3.0 : k == 2 ? 0.5 * a.dt : a.dt);
        T acc[CPT][NE];
#pragma unroll
        for (int c = 0; c < CPT; ++c) {
          const T Vp = Vq[iq[c]], F = Fq[iq[c]], vp = Vp * Pp[ip[c]], vc = Vp * cbp;
#pragma unroll
          for (int e = 0; e < NE; ++e) {
            const T u = e + 1 < NE ? z[c][e + 1 < NE ? e + 1 : 0] : T(0), d = e > 0 ? z[c][e > 0 ? e - 1 : 0] : T(0);
            acc[c][e] = vp * (tc[e] * d - bm * u) - dmp[e] * z[c][e];
            if (live[c] && e < ne) {
              Z[e * arr + iq[c] * RS + ip[c]] = z[c][e];
              Y[e * arr + ip[c] * RS + iq[c]] = F * z[c][e] + vc * (u + cc[e] * d);
            }
          }
        }
        __syncthreads();
        // the q lines, then the p lines, 64 to a wave
        for (int v = w; v < wq + wpn; v += nw) {
          const bool ql = v < wq;
          const int l = (ql ? v : v - wq) * 64 + lane;
          const int len = ql ? a.Np : a.Nq;  // lines per element
          const int e = l / len;
          if (l < (ql ? nql : npl)) stream_line<T, NB>((ql ? Z : Y) + e * arr + (l - e * len), RS, ql ? a.Nq : a.Np);
        }
        __syncthreads();
#pragma unroll
        for (int c = 0; c < CPT; ++c) {
          const T kq = Kp[ip[c]];
#pragma unroll
          for (int e = 0; e < NE; ++e)
            if (live[c] && e < ne) {
              const T k1 = acc[c][e] + (kq * Z[e * arr + iq[c] * RS + ip[c]] + Y[e * arr + ip[c] * RS + iq[c]]);
              z[c][e] = y[c][e] + cst * k1;  // z = y + c k
              if (k == 3) y[c][e] = z[c][e];
            }
        }
        __syncthreads();  // every column has read the arrays
      }
    }
    if (R) {
      double v = 0.0;
#pragma unroll
      for (int c = 0; c < CPT; ++c)
        if (live[c]) v += Cw[iq[c]] * wp[ip[c]] * double(y[c][0]);
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
      if (lane == 0) part[w] = v;
      __syncthreads();
      if (tid == 0) {
        double t = 0.0;
        for (int i = 0; i < nw; ++i) t += part[i];
        R[s * a.ostride + (long long)blockIdx.x * a.bstride] = a.dV * t;
      }
      __syncthreads();
    }
  }
#pragma unroll
  for (int c = 0; c < CPT; ++c)
#pragma unroll
    for (int e = 0; e < NE; ++e)
      if (live[c] && e < ne) st[(long long)e * cols + tid + c * (int)blockDim.x] = y[c][e];
}

}  // namespace chfpe
