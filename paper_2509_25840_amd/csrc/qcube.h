// k_qcube (three modes, grid basis): all three q derivatives of a stage and its
// update in one pass.
//
// A task is one (branch, element) and one run of c = 64 bytes of consecutive p
// points, with the whole q cube: thread (q_2, q_3, part) holds the q_1 lines of
// 16 bytes of p points.  The q_1 planes pass in rounds of PR: X goes to two LDS
// tiles, whose q_2 and q_3 lines a lane each solves; the results s and the q_1
// field G = -(p_1/m_1) X fold into the rows of A t' = A s + B G (as in
// k_pcube_s), so that neither X nor s is kept.  After the last plane a back
// substitution gives t' = s + A^{-1} B G, and the stage update reads t, its
// base state and writes.  The separate (q_2, q_3) and q_1 passes moved seven
// states a stage; this moves four.  Per stage of z = y + c L z, the two passes
// and this: 16^6 FP64 1.84 -> 1.40 ms, FP32 (8 states) 7.3 -> 4.9 ms; 12^6 FP64
// 0.316 -> 0.238 ms, FP32 (8 states) 1.32 -> 0.88 ms.  It reaches 3.8 (FP64) and
// 4.4 TB/s: a run's 64-byte rows halve the use of a cache line per request, and
// one workgroup of 16 waves (two of nine at 12 points) alternates between the
// planes' rounds and the streaming at the end.  Whole RK4 steps with the two
// passes and with this, 12^3 p points, four elements, FP64 and four FP32 states: 5^3 109
// and 72 us, 177 and 109; 7^3 167 132, 304 225; 10^3 384 304, 844 762; 13^3 890
// 830, 2064 1671; 15^3 1417 1383, 3126 2530; 16^3 1729 1660, 3783 3090.
#pragma once

#include "wave.h"

namespace chfpe {

struct QCube {
  int nchunk;  // runs of c p points
  int ntasks, nblk;
};

constexpr int kQcParts = 4;  // 16-byte parts of a run
constexpr int qcube_c(const int tsize) { return kQcParts * 16 / tsize; }
// Planes of a round (the last one takes what is left): the q_1 rows of 14 to 16
// points take most of the 128 registers a thread of 13 to 16 waves has.
constexpr int qcube_planes(const int nb) { return nb >= 14 ? 2 : 4; }
// Rows of the LDS tiles: c values per point and a pad of one point, so that
// rows start in different banks.
__host__ __device__ constexpr int qcube_row(const int n, const int c) { return (n + 1) * c; }
constexpr size_t qcube_lds_vals(const int nb, const int c) {
  return (size_t)2 * qcube_planes(nb) * nb * qcube_row(nb, c) + 3 * (size_t)c;
}

// T: type of the states and of the arithmetic.  NB: points of every q axis (5 to 16).
// epi: the stage update (an Epi, uniform).
template <typename T, int NB>
__global__ void __launch_bounds__(NB * NB * kQcParts)
k_qcube(const Geom g, const Tabs tb, const QCube qc, const T *__restrict__ X, const T *__restrict__ Tacc,
        const T *__restrict__ y, T *__restrict__ xo, const double cst, const int epi) {
  constexpr int V = 16 / (int)sizeof(T);
  constexpr int C = qcube_c(sizeof(T));
  constexpr int PR = qcube_planes(NB);
  constexpr int NR = (NB + PR - 1) / PR;
  constexpr T third = T(1.0 / 3.0);
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int task = xcd_task(blockIdx.x, qc.nblk);
  if (task >= qc.ntasks) return;
  constexpr int plane = NB * NB, row = qcube_row(NB, C), slot = NB * row;
  T *A = reinterpret_cast<T *>(smem_raw);  // [PR][q2][q3][p]
  T *B = A + PR * slot;                    // [PR][q3][q2][p]
  T *K = B + PR * slot;                    // -p_s/m_s (times cb, see wave_rhs) of the run's points, [3][C]
  const int chunk = task % qc.nchunk;      // neighbouring runs share cache lines
  const int ea = task / qc.nchunk;
  const int tid = threadIdx.x;
  const int part = tid % kQcParts, pt = tid / kQcParts;
  const int p0 = chunk * C + part * V;
  const bool own = p0 < g.P;  // (plane * kQcParts threads)
  const int q2 = pt / NB, q3 = pt - q2 * NB;
  const long long eb = (long long)ea * g.E;
  const T *Xe = X + eb;
  auto get = [&](const T *p, const uint32_t at) {
    return *reinterpret_cast<const Vec<T, V> *>(reinterpret_cast<const char *>(p) + at * (uint32_t)sizeof(T));
  };
  // first value of plane i (lanes without points of their own read the element's first ones)
  auto at = [&](const int i) {
    uint32_t o = (uint32_t)(i * plane);
    asm volatile("" : "+s"(o));  // keeps the loads where they are issued (see k_pwave)
    return own ? (o + (uint32_t)pt) * (uint32_t)g.P + (uint32_t)p0 : 0u;
  };
  Vec<T, V> cur[PR];
#pragma unroll
  for (int k = 0; k < PR; ++k) cur[k] = get(Xe, at(k));
  if (tid < 3 * C) {
    const int s = tid / C, pix = min(chunk * C + tid - s * C, g.P - 1);
    K[tid] = T(-tb.pm[s * kTab + (pix / g.PS[s]) % g.Np[s]] * g.dq_cb[s]);
  }
  __syncthreads();

  T ln[NB][V];  // row j of A t' while it collects its terms, then its forward result
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int v = 0; v < V; ++v) ln[j][v] = T(0);
  // weight of G_i in row j
  auto weight = [](const int j, const int i) {
    return i - j == 1 ? T(28) : j - i == 1 ? T(-28) : i > j ? T(1) : T(-1);
  };
  T *mineA = A + q2 * row + q3 * C + part * V, *mineB = B + q3 * row + q2 * C + part * V;
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const int i0 = r * PR;
#pragma unroll
    for (int k = 0; k < PR; ++k) {
      if (i0 + k >= NB) continue;
      *reinterpret_cast<Vec<T, V> *>(mineA + k * slot) = cur[k];
      *reinterpret_cast<Vec<T, V> *>(mineB + k * slot) = cur[k];
      const int i = i0 + k;
#pragma unroll
      for (int v = 0; v < V; ++v) {  // the q_1 field of plane i
        const T gg = K[part * V + v] * cur[k].v[v];
        if (i >= 1) ln[i >= 1 ? i - 1 : 0][v] += weight(i - 1, i) * gg;
        if (i >= 2) ln[i >= 2 ? i - 2 : 0][v] += weight(i - 2, i) * gg;
        if (i + 1 < NB) ln[i + 1 < NB ? i + 1 : 0][v] += weight(i + 1, i) * gg;
        if (i + 2 < NB) ln[i + 2 < NB ? i + 2 : 0][v] += weight(i + 2, i) * gg;
      }
    }
    if (r + 1 < NR) {  // in flight during the line solves
#pragma unroll
      for (int k = 0; k < PR; ++k)
        if (i0 + PR + k < NB) cur[k] = get(Xe, at(i0 + PR + k));
    }
    __syncthreads();
    // q_2 lines of A (fixed plane, q_3, p), q_3 lines of B (fixed plane, q_2, p)
    constexpr int per = NB * C;  // lines of a plane
    const int nA = min(PR, NB - i0) * per;  // and of a field
    for (int l = tid; l < 2 * nA; l += blockDim.x) {
      const int lb = l < nA ? l : l - nA, k = lb / per;
      T *G = (l < nA ? A : B) + k * slot + (lb - k * per);
      if constexpr (NB >= 16 && sizeof(T) == 8)  // the q_1 rows leave no registers for a whole line
        stream_line<T, NB>(G, row, NB);
      else
        wave_line<T, NB, true, false>(G, row, NB, true, nullptr);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PR; ++k) {
      const int i = i0 + k < NB ? i0 + k : 0;
      if (i0 + k >= NB) continue;
      const Vec<T, V> a = *reinterpret_cast<const Vec<T, V> *>(mineA + k * slot);
      const Vec<T, V> b = *reinterpret_cast<const Vec<T, V> *>(mineB + k * slot);
#pragma unroll
      for (int v = 0; v < V; ++v) {
        const T s = K[C + part * V + v] * a.v[v] + K[2 * C + part * V + v] * b.v[v];
        ln[i][v] += s;  // A s
        if (i >= 1) ln[i >= 1 ? i - 1 : 0][v] += third * s;
        if (i + 1 < NB) ln[i + 1 < NB ? i + 1 : 0][v] += third * s;
      }
    }
    // rows up to i - 2 of the round's last plane i are complete
#pragma unroll
    for (int k = 0; k < PR; ++k) {
      const int j = i0 + k - 2;
      if (j < 0 || j >= NB - 2) continue;
#pragma unroll
      for (int v = 0; v < V; ++v)
        ln[j >= 0 ? j : 0][v] = j == 0 ? ln[0][v]
                                       : fma_t(T(-kThomas.inv[j >= 0 ? j : 0] / 3.0), ln[j >= 1 ? j - 1 : 0][v],
                                               ln[j >= 0 ? j : 0][v] * T(kThomas.inv[j >= 0 ? j : 0]));
    }
    __syncthreads();  // the next round overwrites the tiles
  }
  // the rows the last round left
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    if (j < NB - 2) continue;
#pragma unroll
    for (int v = 0; v < V; ++v)
      ln[j][v] = j == 0 ? ln[0][v]
                        : fma_t(T(-kThomas.inv[j] / 3.0), ln[j >= 1 ? j - 1 : 0][v], ln[j][v] * T(kThomas.inv[j]));
  }
  if (!own) return;
  // back substitution and stage update: out = base + cst (t + t'); EPI_OUT: t + t' itself
  const T cs = epi == EPI_OUT ? T(1) : T(cst);
  const T *Te = Tacc + eb;
  T *Oe = xo + eb;
  const T *Be = epi == EPI_H1 ? Xe : epi == EPI_H2 ? y + eb : Oe;
  constexpr int GE = NB >= 14 ? 2 : 4;  // rows of loads issued one group ahead
  T x[V];
#pragma unroll
  for (int v = 0; v < V; ++v) x[v] = T(0);
  Vec<T, V> ct[GE], cb[GE], nt[GE], nb[GE];
  auto load_e = [&](const int j0, Vec<T, V> (&t)[GE], Vec<T, V> (&b)[GE]) {  // rows j0, j0 - 1, ...
#pragma unroll
    for (int k = 0; k < GE; ++k) {
      if (j0 - k < 0) continue;
      const uint32_t o = at(j0 - k);
      t[k] = get(Te, o);
      b[k] = epi == EPI_OUT ? Vec<T, V>{} : get(Be, o);
    }
  };
  load_e(NB - 1, ct, cb);
#pragma unroll
  for (int j0 = NB - 1; j0 >= 0; j0 -= GE) {
    if (j0 >= GE) load_e(j0 - GE, nt, nb);
#pragma unroll
    for (int k = 0; k < GE; ++k) {
      const int j = j0 - k >= 0 ? j0 - k : 0;
      if (j0 - k < 0) continue;
      Vec<T, V> o;
#pragma unroll
      for (int v = 0; v < V; ++v) {
        x[v] = ln[j][v] - T(kThomas.cp[j]) * x[v];
        o.v[v] = cb[k].v[v] + cs * (ct[k].v[v] + x[v]);
      }
      *reinterpret_cast<Vec<T, V> *>(reinterpret_cast<char *>(Oe) + at(j) * (uint32_t)sizeof(T)) = o;
    }
#pragma unroll
    for (int k = 0; k < GE; ++k) {
      ct[k] = nt[k];
      cb[k] = nb[k];
    }
  }
}

}  // namespace chfpe
