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

// Discrete Fourier sums of the spectra, Eqs. (1DIR_Raman) and (2DThz_Raman),
// rectangle rule with weight 1 at t = 0.  Twiddles exp(sign 2 pi i k j / n)
// use the exact reduction (k j mod n) / n before sincospi.
//   out[row][k] = sum_j exp(sign 2 pi i k j / n) in[row][j]   (complex in/out)
__global__ void __launch_bounds__(256)
k_dft_rows(const double2 *__restrict__ in, double2 *__restrict__ out, const int rows, const int n,
           const int in_stride, const int in_step, const int out_stride, const int out_step,
           const double sign) {
  const long long id = (long long)blockIdx.x * 256 + threadIdx.x;
  if (id >= (long long)rows * n) return;
  const int row = (int)(id / n);
  const int k = (int)(id - (long long)row * n);
  double re = 0.0, im = 0.0;
  for (int j = 0; j < n; ++j) {
    const long long kj = ((long long)k * j) % n;
    double sv, cv;
    sincospi(2.0 * (double)kj / (double)n, &sv, &cv);
    sv *= sign;
    const double2 v = in[(long long)row * in_stride + (long long)j * in_step];
    re += v.x * cv - v.y * sv;
    im += v.x * sv + v.y * cv;
  }
  out[(long long)row * out_stride + (long long)k * out_step] = make_double2(re, im);
}

// real input -> complex (imaginary part 0)
__global__ void __launch_bounds__(256)
k_to_complex(const double *__restrict__ in, double2 *__restrict__ out, const long long n) {
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i < n) out[i] = make_double2(in[i], 0.0);
}

// I = scale * omega_k * Im(z)  (omega == nullptr: omega_k = 1)
__global__ void __launch_bounds__(256)
k_spectrum_out(const double2 *__restrict__ z, const long long n, const int n_fast, const double scale,
               const double dw, const int with_omega, double *__restrict__ I) {
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const double w = with_omega ? dw * (double)(i % n_fast) : 1.0;
  I[i] = scale * w * z[i].y;
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
