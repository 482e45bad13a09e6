// Reductions, observables, spectra, start states and bandwidth references of
// the gfx950 CHFPE solver (the propagation kernels are in kernels.h and wave.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace chfpe {

// ---------------------------------------------------------------------------
// reductions and small kernels (FP64)
// ---------------------------------------------------------------------------
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// partial[branch][block] = sum over this block's share of element 0 of
// Cw[qlin] * wp[pidx] * W[qlin * P + pidx]   (fixed order for a fixed grid);
// blockIdx.y selects the branch, whose state starts at W + branch * bstride.
template <typename T>
__global__ void __launch_bounds__(256)
k_reduce_w0(const T *__restrict__ W, const double *__restrict__ Cw, const double *__restrict__ wp,
            const int Q, const int P, double *__restrict__ partial, const long long bstride) {
  __shared__ double sh[4];
  W += (long long)blockIdx.y * bstride;
  partial += (long long)blockIdx.y * gridDim.x;
  double s = 0.0;
  const int n = Q * P;
  for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) {
    const int ql = i / P;
    const int pi = i - ql * P;
    s += Cw[ql] * wp[pi] * double(W[i]);
  }
  s = wave_sum(s);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) partial[blockIdx.x] = (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

// out[b * ostride] = scale * sum(partial[b][0..n)), fixed order, one block per branch b.
__global__ void __launch_bounds__(256)
k_reduce_final(const double *__restrict__ partial, const int n, const double scale,
               double *__restrict__ out, const int ostride) {
  __shared__ double sh[4];
  partial += (long long)blockIdx.x * n;
  out += (long long)blockIdx.x * ostride;
  double s = 0.0;
  for (int i = threadIdx.x; i < n; i += 256) s += partial[i];
  s = wave_sum(s);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) out[0] = scale * ((sh[0] + sh[1]) + (sh[2] + sh[3]));
}

// element 0: h_0 = exp(-beta H / 2) = sq[qlin] * sp[pidx] (unnormalised); other elements: 0
template <typename T>
__global__ void __launch_bounds__(256)
k_boltzmann(T *__restrict__ W, const double *__restrict__ sq, const double *__restrict__ sp,
            const int Q, const int P, const long long total) {
  const int n0 = Q * P;
  for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < total;
       i += (long long)gridDim.x * 256) {
    if (i < n0) {
      const int ii = (int)i;
      const int ql = ii / P;
      const int pi = ii - ql * P;
      W[i] = T(sq[ql] * sp[pi]);
    } else {
      W[i] = T(0);
    }
  }
}

// W <- W * sq[qlin] * sp[pidx] (mul != 0) or W / (sq * sp) (mul == 0), every element
template <typename T>
__global__ void __launch_bounds__(256)
k_sym_scale(T *__restrict__ W, const double *__restrict__ sq, const double *__restrict__ sp,
            const int Q, const int P, const long long total, const int mul) {
  const long long E = (long long)Q * P;
  for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < total;
       i += (long long)gridDim.x * 256) {
    const int ii = (int)(i % E);
    const int ql = ii / P;
    const int pi = ii - ql * P;
    const double f = sq[ql] * sp[pi];
    W[i] = mul ? T(double(W[i]) * f) : T(double(W[i]) / f);
  }
}

// W[0 .. n0) *= 1 / (dV * sum), sum read from device memory
template <typename T>
__global__ void __launch_bounds__(256)
k_normalise(T *__restrict__ W, const double *__restrict__ sum, const double dV, const int n0) {
  const double inv = 1.0 / (dV * sum[0]);
  for (int i = blockIdx.x * 256 + threadIdx.x; i < n0; i += gridDim.x * 256)
    W[i] = T(double(W[i]) * inv);
}

// flag[0] = 1 if any value is not finite
template <typename T>
__global__ void __launch_bounds__(256)
k_check_finite(const T *__restrict__ W, const long long n, int *__restrict__ flag) {
  int bad = 0;
  for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n;
       i += (long long)gridDim.x * 256) {
    const double v = double(W[i]);
    bad |= !(v - v == 0.0);
  }
  if (bad) flag[0] = 1;  // benign race: every writer stores 1
}

// Discrete Fourier sums of the spectra, Eqs. (1DIR_Raman), (2DThz_Raman) and
// (noncorrelation), rectangle rule with weight 1 at t = 0.  Twiddles
// exp(2 pi i k j / n) use the exact reduction (k j mod n) / n before sincospi.
// Lengths up to kDftTab take them from a table of the n-th roots in LDS (TAB);
// the sums were bound by one sincospi and one 64-bit remainder per term
// (4000 points: 1.22 ms, now 17 us; 128 x 256: 164 us, now 14).
constexpr int kDftTab = 8192;

// n-th root j (0 <= j < n)
__device__ __forceinline__ double2 dft_root(const int j, const int n) {
  double2 w;
  sincospi(2.0 * (double)j / (double)n, &w.y, &w.x);
  return w;
}

// One-dimensional spectrum, I[k] = tau omega_k Im sum_j exp(+i omega_k t_j) R[j]
// with omega_k = dw k: only the sines are needed.  A workgroup takes kDftK
// outputs, 256 / kDftK threads each (few outputs per workgroup: 4000 points
// then spread over 250 workgroups); partial sums join in a fixed order.
constexpr int kDftK = 16;
template <bool TAB>
__global__ void __launch_bounds__(256)
k_spectrum_1d(const double *__restrict__ R, const int n, const double tau, const double dw, double *__restrict__ I) {
  extern __shared__ __align__(16) double lds_1d[];  // TAB: sines, then R
  double *S = lds_1d, *Rl = lds_1d + n;
  constexpr int L = 256 / kDftK;
  if constexpr (TAB) {
    for (int j = threadIdx.x; j < n; j += 256) {
      S[j] = dft_root(j, n).y;
      Rl[j] = R[j];
    }
    __syncthreads();
  }
  const int l = threadIdx.x % L;
  const int k = blockIdx.x * kDftK + threadIdx.x / L;
  double s = 0.0;
  if (k < n) {
    int at = (int)(((long long)k * l) % n);
    const int step = (int)(((long long)k * L) % n);
    // U terms' reads go out together (one at a time, each waits out the LDS latency)
    constexpr int U = 8;
    int j = l;
    for (; j + (U - 1) * L < n; j += U * L) {
      double x[U], w[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        x[u] = TAB ? Rl[j + u * L] : R[j + u * L];
        w[u] = TAB ? S[at] : dft_root(at, n).y;
        at += step;
        if (at >= n) at -= n;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) s += x[u] * w[u];
    }
    for (; j < n; j += L) {
      s += (TAB ? Rl[j] : R[j]) * (TAB ? S[at] : dft_root(at, n).y);
      at += step;
      if (at >= n) at -= n;
    }
  }
#pragma unroll
  for (int o = L / 2; o > 0; o >>= 1) s += __shfl_xor(s, o, L);
  if (l == 0 && k < n) I[k] = tau * (dw * (double)k) * s;
}

// One axis of a two-dimensional sum: out(l, k) = sum_j exp(sign 2 pi i k j / n)
// in(l, j) for the nl lines l, with in(l, j) at j * nl + l.  The lanes of a
// wave take consecutive lines (contiguous reads, one twiddle), and where there
// are fewer than 64 lines several k; the four waves of a workgroup take a
// quarter of the terms each, joined in a fixed order, in batches whose reads
// go out together (128 x 256 points: 45 us term by term, now 14).  REAL:
// real input.  IMAG: writes scale * Im alone.  Output (l, k) goes to l * n + k,
// which is the next axis's input order.
template <bool REAL, bool IMAG, bool TAB>
__global__ void __launch_bounds__(256)
k_dft_axis(const double *__restrict__ in, double *__restrict__ out, const int nl, const int n, const int lanes_l,
           const double sign, const double scale) {
  extern __shared__ __align__(16) double2 lds_w[];
  __shared__ double2 part[4][64];
  if constexpr (TAB) {
    for (int j = threadIdx.x; j < n; j += 256) lds_w[j] = dft_root(j, n);
    __syncthreads();
  }
  const double2 *zin = reinterpret_cast<const double2 *>(in);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int kpw = 64 / lanes_l;  // lanes_l: a power of two, 1 .. 64
  const long long lblocks = (nl + lanes_l - 1) / lanes_l, tasks = lblocks * ((n + kpw - 1) / kpw);
  const int quarter = (n + 3) / 4, j0 = wave * quarter, j1 = min(n, j0 + quarter);
  for (long long t = blockIdx.x; t < tasks; t += gridDim.x) {
    const int l = (int)(t % lblocks) * lanes_l + lane % lanes_l;
    const int k = (int)(t / lblocks) * kpw + lane / lanes_l;
    double re = 0.0, im = 0.0;
    if (l < nl && k < n) {
      int at = (int)(((long long)k * j0) % n);
      auto term = [&](const double2 z, const double2 w) {
        const double sv = sign * w.y;
        if constexpr (!IMAG) re += REAL ? z.x * w.x : z.x * w.x - z.y * sv;
        im += REAL ? z.x * sv : z.x * sv + z.y * w.x;
      };
      auto fetch = [&](const int j) {
        const long long p = (long long)j * nl + l;
        return REAL ? make_double2(in[p], 0.0) : zin[p];
      };
      auto root = [&]() {
        const double2 w = TAB ? lds_w[at] : dft_root(at, n);
        at += k;
        if (at >= n) at -= n;
        return w;
      };
      constexpr int U = 8;
      int j = j0;
      for (; j + U <= j1; j += U) {
        double2 z[U], w[U];
#pragma unroll
        for (int u = 0; u < U; ++u) z[u] = fetch(j + u);
#pragma unroll
        for (int u = 0; u < U; ++u) w[u] = root();
#pragma unroll
        for (int u = 0; u < U; ++u) term(z[u], w[u]);
      }
      for (; j < j1; ++j) term(fetch(j), root());
    }
    part[wave][lane] = make_double2(re, im);
    __syncthreads();
    if (wave == 0 && l < nl && k < n) {
      const double2 a = part[0][lane], b = part[1][lane], c = part[2][lane], d = part[3][lane];
      const long long o = (long long)l * n + k;
      im = (a.y + b.y) + (c.y + d.y);
      if constexpr (IMAG)
        out[o] = scale * im;
      else
        reinterpret_cast<double2 *>(out)[o] = make_double2((a.x + b.x) + (c.x + d.x), im);
    }
    __syncthreads();  // the next task overwrites the parts
  }
}

// R[j2 * n_t1 + j0 + b] = Rw[j2 * B + b] for b < nb
__global__ void __launch_bounds__(256)
k_scatter_r(const double *__restrict__ Rw, double *__restrict__ R, const int n_t2, const int B, const int nb,
            const int n_t1, const int j0) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n_t2 * nb) return;
  const int j2 = i / nb;
  const int b = i - j2 * nb;
  R[(long long)j2 * n_t1 + j0 + b] = Rw[(long long)j2 * B + b];
}

// Bandwidth references.  k_stream_copy: dst = src in 16-byte vectors;
// k_stream_mix<NS>: dst = the sum of NS sources (pairs of doubles; NS = 0
// writes zeros), the read/write mixes of the streaming passes.  Each thread
// keeps eight vectors per source in flight before it stores, in a
// grid-stride loop over many workgroups per CU.
constexpr int kStreamU = 8;
__global__ void __launch_bounds__(256)
k_stream_copy(uint4 *__restrict__ dst, const uint4 *__restrict__ src, const long long n16) {
  const long long st = (long long)gridDim.x * 256;
  long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  for (; i + (kStreamU - 1) * st < n16; i += kStreamU * st) {
    uint4 v[kStreamU];
#pragma unroll
    for (int u = 0; u < kStreamU; ++u) v[u] = src[i + u * st];
#pragma unroll
    for (int u = 0; u < kStreamU; ++u) dst[i + u * st] = v[u];
  }
  for (; i < n16; i += st) dst[i] = src[i];
}

template <int NS>
__global__ void __launch_bounds__(256)
k_stream_mix(double2 *__restrict__ dst, const double2 *__restrict__ a, const double2 *__restrict__ b,
             const double2 *__restrict__ c, const long long n16) {
  const long long st = (long long)gridDim.x * 256;
  long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  auto sum = [&](const long long j) {
    double2 v = NS >= 1 ? a[j] : double2{0.0, 0.0};
    if (NS >= 2) {
      const double2 w = b[j];
      v.x += w.x;
      v.y += w.y;
    }
    if (NS >= 3) {
      const double2 w = c[j];
      v.x += w.x;
      v.y += w.y;
    }
    return v;
  };
  for (; i + (kStreamU - 1) * st < n16; i += kStreamU * st) {
    double2 v[kStreamU];
#pragma unroll
    for (int u = 0; u < kStreamU; ++u) v[u] = sum(i + u * st);
#pragma unroll
    for (int u = 0; u < kStreamU; ++u) dst[i + u * st] = v[u];
  }
  for (; i < n16; i += st) dst[i] = sum(i);
}

}  // namespace chfpe
