// Wave-plane kernels: one wave owns whole (rows x cols) planes of a task's
// block, so the two derivatives inside a plane need no workgroup barrier.
//
// A plane is N2 x N3 values, point idx = lane + 64 m of it in register slot m
// of the wave (coalesced loads of 64 consecutive values).  The fields the two
// in-plane derivatives act on go to LDS tiles private to the wave, are solved
// along their lines there (split_line / whole_line), and come back in the
// same layout.  LDS instructions of one wave execute in order, so the waves
// of a workgroup drift apart freely: while one waits for its loads, others
// solve.  Only the derivative across planes meets at two barriers per task.
#pragma once

#include "kernels.h"

namespace chfpe {

// Orders this wave's LDS accesses for the compiler (the hardware executes
// them in program order).
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// A uniform value in scalar registers.
__device__ __forceinline__ float uniform(const float x) {
  return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(x)));
}
__device__ __forceinline__ double uniform(const double x) {
  const int lo = __builtin_amdgcn_readfirstlane(__double2loint(x));
  const int hi = __builtin_amdgcn_readfirstlane(__double2hiint(x));
  return __hiloint2double(hi, lo);
}

// Block of `bytes` bytes at p as a buffer: loads past its end return zero
// and move nothing, so a missing hierarchy neighbour is a buffer of no bytes.
// That keeps every load unconditional (a load under a branch is waited for
// where the branch joins) at no traffic.
typedef __amdgpu_buffer_rsrc_t Buf;
__device__ __forceinline__ Buf make_buf(const void *p, const uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00027000);
}
// V consecutive values of type T, moved by one instruction.
template <typename T, int V>
struct alignas(sizeof(T) * V) Vec {
  T v[V];
};
// values at byte offset voff; the instruction's uniform offset stays zero, as
// the intrinsic leaves it out of the comparison with the buffer's size
template <typename T, int V>
__device__ __forceinline__ Vec<T, V> buf_load(const Buf r, const uint32_t voff) {
  if constexpr (sizeof(T) * V == 16)
    return __builtin_bit_cast(Vec<T, V>, __builtin_amdgcn_raw_buffer_load_b128(r, (int)voff, 0, 0));
  else if constexpr (sizeof(T) * V == 8)
    return __builtin_bit_cast(Vec<T, V>, __builtin_amdgcn_raw_buffer_load_b64(r, (int)voff, 0, 0));
  else
    return __builtin_bit_cast(Vec<T, V>, __builtin_amdgcn_raw_buffer_load_b32(r, (int)voff, 0, 0));
}
// Closure weights of one axis in LDS: rows p1, m1, p2, m2 of NB entries (third
// off-diagonals are not used, kClosBands = 2).
constexpr int kWClosRows = 4;
constexpr int wave_clos_vals(const int nb) { return kWClosRows * nb; }

// Right-hand side of the compact scheme at position i, over cb = 1/(36 h):
// ca / cb = (7/9) / (1/36) = 28.  The fields are formed with the factor cb in
// their coefficients; a closure's weights hold 1/h themselves.
template <typename T, int NB, bool CLOS>
__device__ __forceinline__ T wave_rhs(const int i, const T fm2, const T fm1, const T fp1, const T fp2, const T *ct) {
  if constexpr (CLOS)
    return ct[i] * fp1 + ct[NB + i] * fm1 + ct[2 * NB + i] * fp2 + ct[3 * NB + i] * fm2;
  else
    return fma_t(T(28), fp1 - fm1, fp2 - fm2);
}

// Compact derivative of a line of n <= NB values in LDS by one lane, in place
// through registers.  FULL: n = NB; else values past the line are zero, and so
// are the forward results there, so that the sweeps run over NB positions
// with no branch: reads past the line repeat its last value's address, and
// the stores, last position first, end with that value's own.  One lane per line takes six FP64 instructions a value; two
// lanes that meet in the middle halve the chain, but their addresses,
// mirrored operands and exchange doubled the instructions (24^3: 22 k
// instructions per wave against 13 k, at 47% of the VALU).
template <typename T, int NB, bool FULL, bool CLOS>
__device__ __forceinline__ void wave_line(T *G, const int stride, const int n, const bool act, const T *ct) {
  T f[NB];
  const int last = (n - 1) * stride;
  auto at = [&](const int i) { return FULL ? i * stride : min(i * stride, last); };
#pragma unroll
  for (int i = 0; i < NB; ++i) f[i] = G[at(i)];
  if constexpr (!FULL) {
#pragma unroll
    for (int i = 0; i < NB; ++i) f[i] = i < n ? f[i] : T(0);
  }
  T fm2 = T(0), fm1 = T(0), dprev = T(0);
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const T f0 = f[i];
    const T fp1 = i + 1 < NB ? f[i + 1 < NB ? i + 1 : 0] : T(0);
    const T fp2 = i + 2 < NB ? f[i + 2 < NB ? i + 2 : 0] : T(0);
    const T r = wave_rhs<T, NB, CLOS>(i, fm2, fm1, fp1, fp2, ct);
    const T d = i == 0 ? r : fma_t(T(-kThomas.inv[i] / 3.0), dprev, r * T(kThomas.inv[i]));
    fm2 = fm1;
    fm1 = f0;
    dprev = d;
    f[i] = FULL || i < n ? d : T(0);
  }
  T x = T(0);
#pragma unroll
  for (int i = NB - 1; i >= 0; --i) {
    x = f[i] - T(kThomas.cp[i]) * x;
    f[i] = x;
  }
  if (act) {
#pragma unroll
    for (int i = NB - 1; i >= 0; --i) G[at(i)] = f[i];
  }
}

// Compact derivative, over cb (see wave_rhs), of a line of n <= NB values (n
// uniform over the wave) in LDS by one lane.  Streamed:
// a forward result overwrites its value once the sweep's window has read it,
// and the back substitution overwrites it in turn, so that few registers hold
// the line.  Reads run kStreamPF positions ahead (and may touch that many rows
// past the array).  Positions go in blocks of eight with no branch inside but
// in the block the line ends in: with one per position, a step waits for its
// five dependent instructions (100 cycles instead of 35).
constexpr int kStreamPF = 4;
template <typename T, int NB>
__device__ __forceinline__ void stream_line(T *G, const int stride, const int n) {
  constexpr int PF = kStreamPF, BL = 8;
  static_assert(NB % BL == 0, "whole blocks");
  T f[PF + 1];  // f_i .. f_{i + PF}; zero past the line
#pragma unroll
  for (int j = 0; j < PF; ++j) f[j] = G[j * stride];  // lines have at least five values
  T fm1 = T(0), fm2 = T(0), d = T(0);
  auto forward = [&](const int i) {
    const T nx = i + PF < NB ? G[(i + PF < NB ? i + PF : 0) * stride] : T(0);
    f[PF] = i + PF < n ? nx : T(0);
    const T r = fma_t(T(28), f[1] - fm1, f[2] - fm2);
    d = i == 0 ? r : fma_t(T(-kThomas.inv[i] / 3.0), d, r * T(kThomas.inv[i]));
    G[i * stride] = d;
    fm2 = fm1;
    fm1 = f[0];
#pragma unroll
    for (int j = 0; j < PF; ++j) f[j] = f[j + 1];
  };
#pragma unroll
  for (int i0 = 0; i0 < NB; i0 += BL) {
    if (i0 + BL <= n) {
#pragma unroll
      for (int i = i0; i < i0 + BL; ++i) forward(i);
    } else if (i0 < n) {
#pragma unroll
      for (int i = i0; i < i0 + BL - 1; ++i)
        if (i < n) forward(i);
    }
  }
  asm volatile("" ::: "memory");  // the results are read back, not kept
  T x = d, v[PF + 1];  // d_i .. d_{i - PF}
#pragma unroll
  for (int j = 0; j < PF; ++j) v[j] = G[(n - 2 - j) * stride];
  auto backward = [&](const int i) {
    v[PF] = G[(i >= PF ? i - PF : 0) * stride];
    x = v[0] - T(kThomas.cp[i]) * x;
    G[i * stride] = x;
#pragma unroll
    for (int j = 0; j < PF; ++j) v[j] = v[j + 1];
  };
#pragma unroll
  for (int i0 = NB - BL; i0 >= 0; i0 -= BL) {
    if (i0 + BL <= n - 1) {
#pragma unroll
      for (int i = i0 + BL - 1; i >= i0; --i) backward(i);
    } else if (i0 < n - 1) {
#pragma unroll
      for (int i = i0 + BL - 2; i >= i0; --i)
        if (i < n - 1) backward(i);
    }
  }
}

// Both in-plane derivatives of a wave's PS planes, in place: GA ([plane][N2]
// rows of N3) along the rows axis, GB along the columns axis.  GB holds its
// field transposed ([plane][N3] rows of N2), so that a line of either field
// is a column of its tile: the lanes of a row read consecutive words, and
// every address is one base plus constants.
template <typename T, int NB, int PS, bool EXACT, bool CLOS>
__device__ __forceinline__ void plane_solve(T *GA, T *GB, const int lane, const int N2, const int N3, const int rs,
                                            const int slot, const T *ct2, const T *ct3) {
  static_assert(2 * PS * NB <= 64 || (!EXACT && NB <= 32), "a lane per line");
  if constexpr (EXACT) {
    const int l = min(lane, 2 * PS * NB - 1);
    const bool b = l >= PS * NB;
    const int r = b ? l - PS * NB : l;
    const int pl = r / NB;
    wave_line<T, NB, true, CLOS>((b ? GB : GA) + pl * slot + (r - pl * NB), rs, NB, lane < 2 * PS * NB,
                                 b ? ct3 : ct2);
  } else {  // one plane; the lower half of the wave takes GA's lines, the upper half GB's
    const bool b = lane >= 32;
    const int nl = b ? N2 : N3;
    const int c = (lane & 31) < nl ? lane & 31 : 0;
    wave_line<T, NB, false, CLOS>((b ? GB : GA) + c, rs, b ? N3 : N2, (lane & 31) < nl, b ? ct3 : ct2);
  }
}

constexpr int wave_gcd(const int a, const int b) { return b == 0 ? a : wave_gcd(b, a % b); }

// Values a lane moves at a time: 16 bytes for cubes.  A vector memory
// instruction holds a CU's address unit for about 16 cycles whatever its width
// (four lanes a cycle), so one value per lane bounds a block kernel long
// before HBM does: 15 cycles per load and CU at 16^6 in FP32 (eight states:
// 4.1 ms per launch; with 16-byte loads and the line solves below, 3.0 ms).
constexpr int wave_vec(const int tsize, const bool exact) { return exact ? 16 / tsize : 1; }
// Planes a wave takes together (their 2 PS NB lines fill its lanes), groups of
// planes per wave, waves of a workgroup for lines of up to NB points.
constexpr int wave_ps(const int nb, const bool exact) { return !exact ? 1 : nb >= 24 ? 1 : nb >= 12 ? 2 : 4; }
constexpr int pwave_npw(const int nb, const bool exact) { return nb >= 24 ? 3 : !exact ? 4 : nb >= 12 ? 2 : 1; }
constexpr int pwave_waves(const int nb, const bool exact) {
  const int per = wave_ps(nb, exact) * pwave_npw(nb, exact);
  return (nb + per - 1) / per;
}
// Vectors per lane of PS planes of NB x NB points.
constexpr int wave_nv(const int nb, const int ps, const int v) { return (ps * nb * nb + 64 * v - 1) / (64 * v); }
// LDS tiles ([N2][N3], or the transposed field) have an odd row stride:
// lanes along a row and lanes down a column both read distinct banks (128
// bytes a cycle).  The distance of two tiles is chosen for the line solves,
// whose lanes run over the NB columns of PS tiles of each field in turn:
// NB values past a multiple of the banks where PS > 1, so that the tiles of
// one field follow each other's banks, and wave_pad() values between the two
// fields' tiles.
__host__ __device__ constexpr int wave_rs(const int n2, const int n3) { return (n2 > n3 ? n2 : n3) | 1; }
__host__ __device__ constexpr int wave_slot(const int n2, const int n3, const int ps) {
  const int nb = n2 > n3 ? n2 : n3, banks = 32, off = ps > 1 ? nb % banks : 0;
  return (nb * wave_rs(n2, n3) - off + banks - 1) / banks * banks + off;
}
constexpr int wave_pad(const int nb, const int ps) { return ps * nb; }
// Values of the LDS of a k_pwave workgroup of nw waves: a tile per plane, PS
// more per wave, the p grids, and the closure weights.
constexpr size_t pwave_lds_vals(const int nb, const int n1, const int n2, const int n3, const int nw, const int ps,
                                const bool clos) {
  return (size_t)(n1 + nw * ps) * wave_slot(n2, n3, ps) + wave_pad(nb, ps) + 3 * (size_t)nb +
         (clos ? 3 * (size_t)wave_clos_vals(nb) : 0);
}
// Vectors of loads in flight ahead of their use.
constexpr int pwave_depth(const int nv) { return nv < 2 ? 1 : 2; }
// Waves per SIMD the register budget aims at (what the LDS allows: one
// workgroup of eight waves per CU for FP64 lines of 24 points, three of four
// waves for 16).
constexpr int pwave_occ(const int nb, const int tsize) { return nb >= 24 ? 2 : tsize == 4 ? 4 : 3; }

// ---------------------------------------------------------------------------
// k_pwave (three modes): every p derivative and pointwise term of one q point
// ---------------------------------------------------------------------------
// Same task, inputs and result as k_pcube.  Wave w takes the groups w, w + NW,
// ... of PS planes of the p block: loads h_n and its neighbours there, forms
// the three fields, solves the p_2 and p_3 lines in its own tiles and keeps s
// (pointwise, p_2 and p_3 terms) in registers; the p_1 field is left in the
// planes' tiles.  After a barrier the workgroup's threads solve the p_1 lines
// through the tiles in place; after another each wave adds its s and stores.
// Two barriers a task (k_pcube: three a round of planes) let the eight waves
// of a CU drift apart, and 16-byte loads of buffers that are empty where a
// neighbour is missing keep the address unit free.  Per launch, before and
// after: 24^6 FP64 16.2 -> 9.0 ms (3.4 TB/s of algorithmic bytes; its HBM
// traffic is those bytes), 16^6 FP64 1.15 -> 0.68 ms, 16^6 FP32 (8 states)
// 4.28 -> 3.0 ms, 12^6 FP64 0.27 -> 0.156 ms and 0.57 -> 0.184 ms with a
// closure (its weights come from LDS).  At 24^6 the waves now wait for loads
// 42% of their cycles, VALU issue is 27% and the LDS 44% busy: one workgroup
// of eight waves fills the LDS.
// NVR = 0: a cube of NB points on every axis; else a block of axes of at most
// NB points, with planes of at most 64 NVR points.
template <typename T, typename TO, int NB, int NVR, bool PERTURB, bool CLOS = false>
__global__ void __launch_bounds__((64 * pwave_waves(NB, NVR == 0)), (pwave_occ(NB, sizeof(T))))
k_pwave(const Geom g, const Tabs tb, const PCube pc, const T *__restrict__ X, TO *__restrict__ out,
        const double *__restrict__ grad) {
  constexpr bool EXACT = NVR == 0;
  constexpr int V = wave_vec(sizeof(T), EXACT);
  constexpr int PS = wave_ps(NB, EXACT);
  constexpr int NV = EXACT ? wave_nv(NB, PS, V) : NVR;
  constexpr int NPW = pwave_npw(NB, EXACT);
  constexpr int DEPTH = pwave_depth(NV);
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int task = xcd_task(blockIdx.x, pc.nblk);
  if (task >= pc.ntasks) return;
  const int N1 = EXACT ? NB : pc.N1, N2 = EXACT ? NB : pc.N2, N3 = EXACT ? NB : pc.N3;
  const int plane = EXACT ? NB * NB : pc.plane;
  const int rs = wave_rs(N2, N3);
  const int slot = wave_slot(N2, N3, PS);
  const int nw = EXACT ? pwave_waves(NB, EXACT) : (int)(blockDim.x >> 6);
  T *tiles = reinterpret_cast<T *>(smem_raw);     // [N1][slot]
  T *own = tiles + N1 * slot + wave_pad(NB, PS);  // [nw][PS][slot]
  T *P1 = own + nw * PS * slot, *P2 = P1 + NB, *P3 = P2 + NB;
  T *ctab = P3 + NB;  // closure weights [3][4][NB]
  const int ne_all = g.ne * g.nbatch;
  const int ea = task % ne_all;  // (branch, element): elements of one q point are adjacent tasks
  const int ql = task / ne_all;
  const int br = ea / g.ne;
  const int e = ea - br * g.ne;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int Q = g.Q;

  const long long blk = (long long)ql * g.P;
  const uint32_t bytes = (uint32_t)g.P * (uint32_t)sizeof(T);
  const T *Xb = X + (long long)br * g.ne * g.E + blk;
  const Buf bh = make_buf(X + (long long)ea * g.E + blk, bytes);
  Buf bu[3], bd[3];
  // fields (times cb, see wave_rhs): F_s h + vu u + vd d; pointwise: p_s (pwd d - pwu u)
  T Fv[3], vu[3], vd[3], pwu[3], pwd[3], xs[3];
  bool any_up = false;
#pragma unroll
  for (int s = 0; s < 3; ++s) {
    const int up = PERTURB ? -1 : tb.up[e * 3 + s];
    const int dn = PERTURB ? -1 : tb.dn[e * 3 + s];
    const double cb = CLOS ? 1.0 : g.dp_cb[s];
    any_up = any_up || up >= 0;
    bu[s] = make_buf(Xb + (long long)max(up, 0) * g.E, up >= 0 ? bytes : 0);
    bd[s] = make_buf(Xb + (long long)max(dn, 0) * g.E, dn >= 0 ? bytes : 0);
    if (PERTURB) {
      const double gr = grad[s * Q + ql];
      Fv[s] = uniform(T(gr * cb));
      xs[s] = uniform(T(gr * g.bm[s]));  // times p_s
      vu[s] = vd[s] = pwu[s] = pwd[s] = T(0);
    } else {
      const double vp = tb.VpQ[s * Q + ql];
      Fv[s] = uniform(T(tb.F[s * Q + ql] * cb));
      vu[s] = uniform(T(vp * cb));
      vd[s] = uniform(T(vp * tb.cc[e * 3 + s] * cb));
      pwd[s] = uniform(T(vp * 0.5 * tb.tc[e * 3 + s]));
      pwu[s] = uniform(T(vp * g.bm[s]));
      xs[s] = T(0);
    }
  }
  const T dmp = PERTURB ? T(0) : uniform(T(tb.damp[e]));

  // the p grids and closure weights come to LDS; their loads go out before
  // the first loads of the planes, the stores follow those
  const int tl = min(tid, NB - 1);
  const T tp1 = T(tb.pg[tl]), tp2 = T(tb.pg[1 * kTab + tl]), tp3 = T(tb.pg[2 * kTab + tl]);
  auto fill_tables = [&]() {
    if (tid < NB) {
      P1[tid] = tp1;
      P2[tid] = tp2;
      P3[tid] = tp3;
    }
    if constexpr (CLOS) {
      for (int v = tid; v < 3 * wave_clos_vals(NB); v += blockDim.x) {
        const int ax = v / wave_clos_vals(NB), r = v - ax * wave_clos_vals(NB);
        ctab[v] = T(tb.clos[(g.M + ax) * 2 * kClosRows * kTab + (r / NB) * kTab + r % NB]);
      }
    }
    __syncthreads();
  };
  const T *ct1 = ctab, *ct2 = ctab + wave_clos_vals(NB), *ct3 = ct2 + wave_clos_vals(NB);

  // Vector m of this lane: V consecutive points, in one row, from point
  // V (lane + 64 m) of the group's PS planes.  The pattern repeats every PER
  // vectors, DR rows further down, so only PER of each are kept.
  constexpr int PER0 = NB / V / wave_gcd(NB / V, 64);
  constexpr int DR = 64 * V * PER0 / NB;
  constexpr bool REP = EXACT && PER0 < NV && PS == 1;
  constexpr int PER = REP ? PER0 : NV;
  int row[PER], col[PER], pln[PER];
#pragma unroll
  for (int m = 0; m < PER; ++m) {
    const int idx = min(V * (lane + 64 * m), PS * plane - V);
    pln[m] = PS > 1 ? idx / plane : 0;
    const int in = idx - pln[m] * plane;
    row[m] = in / N3;
    col[m] = in - row[m] * N3;
  }
  // its place in GA's tiles, and in GB's (transposed)
  auto at_a = [&](const int m) { return pln[m % PER] * slot + row[m % PER] * rs + col[m % PER] + m / PER * (DR * rs); };
  auto at_b = [&](const int m) { return pln[m % PER] * slot + col[m % PER] * rs + row[m % PER] + m / PER * DR; };
  auto mine = [&](const int m) {
    return (EXACT && V * 64 * (m + 1) <= PS * NB * NB) || V * (lane + 64 * m) < PS * plane;
  };

  struct In {
    Vec<T, V> h, u[3], d[3];
  };
  T sv[NPW][NV][V];
  auto sweep = [&](auto UP) {
    constexpr bool up = decltype(UP)::value;
    // The plane offset passes through an empty asm statement each time: the
    // buffers are read-only, and without it every load of the kernel may be
    // hoisted to the top.  It is part of the offset per lane, the one that is
    // compared with the buffer's size.
    auto load = [&](const int k, const int m) {
      In x;
      uint32_t so = (uint32_t)((w + k * nw) * (PS * plane)) * (uint32_t)sizeof(T);
      asm volatile("" : "+s"(so));
      const uint32_t vo = so + (uint32_t)(lane + 64 * m) * (uint32_t)(V * sizeof(T));
      x.h = buf_load<T, V>(bh, vo);
      if constexpr (!PERTURB) {
#pragma unroll
        for (int s = 0; s < 3; ++s) {
          if constexpr (up) x.u[s] = buf_load<T, V>(bu[s], vo);
          x.d[s] = buf_load<T, V>(bd[s], vo);
        }
      }
      return x;
    };
    // vector v = k NV + m of the wave goes to ring[v % DEPTH]; loads run DEPTH
    // ahead, so those of the next group are in flight during the line solves
    In ring[DEPTH];
#pragma unroll
    for (int v = 0; v < DEPTH && v < NPW * NV; ++v) ring[v] = load(v / NV, v % NV);
    fill_tables();
#pragma unroll
    for (int k = 0; k < NPW; ++k) {
      const int i0 = (w + k * nw) * PS;
      if (!EXACT && i0 >= N1) break;  // uniform over the wave
      Vec<T, V> g1[NV];
      T *GA = tiles + i0 * slot, *GB = own + w * PS * slot;
#pragma unroll
      for (int m = 0; m < NV; ++m) {
        const int v = k * NV + m;
        const In cur = ring[v % DEPTH];
        const T p1 = P1[i0 + pln[m % PER]];
        const T p2 = P2[row[m % PER] + m / PER * DR];
        Vec<T, V> f2, f3;
#pragma unroll
        for (int q = 0; q < V; ++q) {
          const T h = cur.h.v[q], p3 = P3[col[m % PER] + q];
          T s, a1 = Fv[0] * h, a2 = Fv[1] * h, a3 = Fv[2] * h;
          if constexpr (PERTURB) {
            s = -(xs[0] * p1 + xs[1] * p2 + xs[2] * p3) * h;
          } else {
            const T d1 = cur.d[0].v[q], d2 = cur.d[1].v[q], d3 = cur.d[2].v[q];
            T t1 = pwd[0] * d1, t2 = pwd[1] * d2, t3 = pwd[2] * d3;
            a1 += vd[0] * d1;
            a2 += vd[1] * d2;
            a3 += vd[2] * d3;
            if constexpr (up) {
              const T u1 = cur.u[0].v[q], u2 = cur.u[1].v[q], u3 = cur.u[2].v[q];
              t1 -= pwu[0] * u1;
              t2 -= pwu[1] * u2;
              t3 -= pwu[2] * u3;
              a1 += vu[0] * u1;
              a2 += vu[1] * u2;
              a3 += vu[2] * u3;
            }
            s = -dmp * h + p1 * t1 + p2 * t2 + p3 * t3;
          }
          asm volatile("" : "+v"(s), "+v"(a1));  // formed here: their inputs are not kept
          sv[k][m][q] = s;
          g1[m].v[q] = a1;
          f2.v[q] = a2;
          f3.v[q] = a3;
        }
        if (v + DEPTH < NPW * NV) ring[v % DEPTH] = load((v + DEPTH) / NV, (v + DEPTH) % NV);  // (past the block: zeros, unused)
        if (mine(m)) {
#pragma unroll
          for (int q = 0; q < V; ++q) GA[at_a(m) + q] = f2.v[q];
#pragma unroll
          for (int q = 0; q < V; ++q) GB[at_b(m) + q * rs] = f3.v[q];
        }
      }
      wave_lds_fence();
      plane_solve<T, NB, PS, EXACT, CLOS>(GA, GB, lane, N2, N3, rs, slot, ct2, ct3);
      wave_lds_fence();
#pragma unroll
      for (int m = 0; m < NV; ++m) {
        if (!mine(m)) continue;
#pragma unroll
        for (int q = 0; q < V; ++q) sv[k][m][q] += GA[at_a(m) + q] + GB[at_b(m) + q * rs];
      }
      wave_lds_fence();
#pragma unroll
      for (int m = 0; m < NV; ++m) {
        if (!mine(m)) continue;
#pragma unroll
        for (int q = 0; q < V; ++q) GA[at_a(m) + q] = g1[m].v[q];
      }
    }
  };
  if (!PERTURB && any_up)  // uniform: the elements below the hierarchy's last level
    sweep(std::true_type{});
  else
    sweep(std::false_type{});
  __syncthreads();
  // p_1 lines, one per thread, in place in the tiles
  for (int l = tid; l < plane; l += blockDim.x) {
    const int r2 = l / N3;
    wave_line<T, NB, EXACT, CLOS>(tiles + r2 * rs + (l - r2 * N3), slot, N1, true, ct1);
  }
  __syncthreads();
  TO *Oe = out + (long long)ea * g.E + blk;
#pragma unroll
  for (int k = 0; k < NPW; ++k) {
    const int i0 = (w + k * nw) * PS;
    if (!EXACT && i0 >= N1) break;
#pragma unroll
    for (int m = 0; m < NV; ++m)
      if (mine(m)) {
        const T *a = tiles + i0 * slot + at_a(m);
        Vec<TO, V> o;
#pragma unroll
        for (int q = 0; q < V; ++q) o.v[q] = TO(sv[k][m][q] + a[q]);
        *reinterpret_cast<Vec<TO, V> *>(reinterpret_cast<char *>(Oe) +
                                        (uint32_t)(i0 * plane + V * (lane + 64 * m)) * (uint32_t)sizeof(TO)) = o;
      }
  }
}

// ---------------------------------------------------------------------------
// k_pwave2 (two modes): the p side of one q point by one wave
// ---------------------------------------------------------------------------
// Same task, inputs and result as k_pblock for two modes, in the wave-plane
// form: the p block of a task is one (p_1, p_2) plane, a wave takes a task by
// itself (four consecutive tasks, elements of one q point, per workgroup),
// and there is no barrier but the one after the grids are in LDS.  Loads of a
// missing neighbour are of an empty buffer.  Per launch, before (k_pblock:
// one-value loads and three barriers a task) and after: 32^4 with 64 FP64
// states 3.58 -> 2.45 ms (4.4 TB/s of algorithmic bytes), 64 FP32 states 2.17
// -> 1.22 ms; one FP64 state of 32^4 0.054 -> 0.042, 24^4 0.024 -> 0.017,
// 27 x 28 points 0.072 -> 0.044, 16^4 0.011 -> 0.009 ms.
constexpr int kPWave2Waves = 4;
constexpr size_t pwave2_lds_vals(const int nb, const int n1, const int n2, const bool clos) {
  return 2 * (size_t)kPWave2Waves * (wave_slot(n1, n2, 1) + 16) + 2 * (size_t)nb +
         (clos ? 2 * (size_t)wave_clos_vals(nb) : 0);
}

template <typename T, typename TO, int NB, int NVR, bool PERTURB, bool CLOS = false>
__global__ void __launch_bounds__(64 * kPWave2Waves)
k_pwave2(const Geom g, const Tabs tb, const PCube pc, const T *__restrict__ X, TO *__restrict__ out,
         const double *__restrict__ grad) {
  constexpr bool EXACT = NVR == 0;
  constexpr int V = wave_vec(sizeof(T), EXACT);
  constexpr int NV = EXACT ? wave_nv(NB, 1, V) : NVR;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wg = xcd_task(blockIdx.x, pc.nblk);
  if (wg * kPWave2Waves >= pc.ntasks) return;
  const int task = min(wg * kPWave2Waves + w, pc.ntasks - 1);  // (waves past the last task store nothing)
  const int N2 = EXACT ? NB : pc.N2, N3 = EXACT ? NB : pc.N3;
  const int plane = EXACT ? NB * NB : pc.plane;
  const int rs = wave_rs(N2, N3), slot = wave_slot(N2, N3, 1);
  T *GA = reinterpret_cast<T *>(smem_raw) + 2 * w * (slot + 16), *GB = GA + slot + 16;
  T *P1 = reinterpret_cast<T *>(smem_raw) + 2 * kPWave2Waves * (slot + 16), *P2 = P1 + NB;
  T *ctab = P2 + NB;
  const int ne_all = g.ne * g.nbatch;
  const int ea = task % ne_all;
  const int ql = task / ne_all;
  const int br = ea / g.ne;
  const int e = ea - br * g.ne;
  const int Q = g.Q;

  const long long blk = (long long)ql * g.P;
  const uint32_t bytes = (uint32_t)g.P * (uint32_t)sizeof(T);
  const T *Xb = X + (long long)br * g.ne * g.E + blk;
  const Buf bh = make_buf(X + (long long)ea * g.E + blk, bytes);
  Buf bu[2], bd[2];
  // fields (times cb, see wave_rhs) and pointwise factors, as in k_pwave
  T Fv[2], vu[2], vd[2], pwu[2], pwd[2], xs[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const int up = PERTURB ? -1 : tb.up[e * 3 + s];
    const int dn = PERTURB ? -1 : tb.dn[e * 3 + s];
    const double cb = CLOS ? 1.0 : g.dp_cb[s];
    bu[s] = make_buf(Xb + (long long)max(up, 0) * g.E, up >= 0 ? bytes : 0);
    bd[s] = make_buf(Xb + (long long)max(dn, 0) * g.E, dn >= 0 ? bytes : 0);
    if (PERTURB) {
      const double gr = grad[s * Q + ql];
      Fv[s] = uniform(T(gr * cb));
      xs[s] = uniform(T(gr * g.bm[s]));
      vu[s] = vd[s] = pwu[s] = pwd[s] = T(0);
    } else {
      const double vp = tb.VpQ[s * Q + ql];
      Fv[s] = uniform(T(tb.F[s * Q + ql] * cb));
      vu[s] = uniform(T(vp * cb));
      vd[s] = uniform(T(vp * tb.cc[e * 3 + s] * cb));
      pwd[s] = uniform(T(vp * 0.5 * tb.tc[e * 3 + s]));
      pwu[s] = uniform(T(vp * g.bm[s]));
      xs[s] = T(0);
    }
  }
  const T dmp = PERTURB ? T(0) : uniform(T(tb.damp[e]));
  const int tl = min(tid, NB - 1);
  const T tp1 = T(tb.pg[tl]), tp2 = T(tb.pg[kTab + tl]);

  constexpr int PER0 = NB / V / wave_gcd(NB / V, 64);
  constexpr int DR = 64 * V * PER0 / NB;
  constexpr int PER = EXACT && PER0 < NV ? PER0 : NV;
  int row[PER], col[PER];
#pragma unroll
  for (int m = 0; m < PER; ++m) {
    const int idx = min(V * (lane + 64 * m), plane - V);
    row[m] = idx / N3;
    col[m] = idx - row[m] * N3;
  }
  auto at_a = [&](const int m) { return row[m % PER] * rs + col[m % PER] + m / PER * (DR * rs); };
  auto at_b = [&](const int m) { return col[m % PER] * rs + row[m % PER] + m / PER * DR; };
  auto mine = [&](const int m) { return (EXACT && V * 64 * (m + 1) <= NB * NB) || V * (lane + 64 * m) < plane; };

  struct In {
    Vec<T, V> h, u[2], d[2];
  };
  auto load = [&](const int m) {
    In x;
    uint32_t vo = (uint32_t)(lane + 64 * m) * (uint32_t)(V * sizeof(T));
    asm volatile("" : "+v"(vo));  // keeps the loads where they are issued (see k_pwave)
    x.h = buf_load<T, V>(bh, vo);
    if constexpr (!PERTURB) {
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        x.u[s] = buf_load<T, V>(bu[s], vo);
        x.d[s] = buf_load<T, V>(bd[s], vo);
      }
    }
    return x;
  };
  constexpr int DEPTH = NV < 3 ? NV : 3;
  In ring[DEPTH];
#pragma unroll
  for (int m = 0; m < DEPTH; ++m) ring[m] = load(m);
  if (tid < NB) {
    P1[tid] = tp1;
    P2[tid] = tp2;
  }
  if constexpr (CLOS) {
    for (int v = tid; v < 2 * wave_clos_vals(NB); v += blockDim.x) {
      const int ax = v / wave_clos_vals(NB), r = v - ax * wave_clos_vals(NB);
      ctab[v] = T(tb.clos[(g.M + ax) * 2 * kClosRows * kTab + (r / NB) * kTab + r % NB]);
    }
  }
  __syncthreads();
  T sv[NV][V];
#pragma unroll
  for (int m = 0; m < NV; ++m) {
    const In cur = ring[m % DEPTH];
    const T p1 = P1[row[m % PER] + m / PER * DR];
    Vec<T, V> f1, f2;
#pragma unroll
    for (int q = 0; q < V; ++q) {
      const T h = cur.h.v[q], p2 = P2[col[m % PER] + q];
      T s, a1 = Fv[0] * h, a2 = Fv[1] * h;
      if constexpr (PERTURB) {
        s = -(xs[0] * p1 + xs[1] * p2) * h;
      } else {
        const T u1 = cur.u[0].v[q], u2 = cur.u[1].v[q], d1 = cur.d[0].v[q], d2 = cur.d[1].v[q];
        a1 += vd[0] * d1 + vu[0] * u1;
        a2 += vd[1] * d2 + vu[1] * u2;
        s = -dmp * h + p1 * (pwd[0] * d1 - pwu[0] * u1) + p2 * (pwd[1] * d2 - pwu[1] * u2);
      }
      asm volatile("" : "+v"(s));  // formed here: its inputs are not kept
      sv[m][q] = s;
      f1.v[q] = a1;
      f2.v[q] = a2;
    }
    if (m + DEPTH < NV) ring[m % DEPTH] = load(m + DEPTH);
    if (mine(m)) {
#pragma unroll
      for (int q = 0; q < V; ++q) GA[at_a(m) + q] = f1.v[q];
#pragma unroll
      for (int q = 0; q < V; ++q) GB[at_b(m) + q * rs] = f2.v[q];
    }
  }
  wave_lds_fence();
  plane_solve<T, NB, 1, EXACT, CLOS>(GA, GB, lane, N2, N3, rs, slot, ctab, ctab + wave_clos_vals(NB));
  wave_lds_fence();
  if (wg * kPWave2Waves + w >= pc.ntasks) return;
  TO *Oe = out + (long long)ea * g.E + blk;
#pragma unroll
  for (int m = 0; m < NV; ++m) {
    if (!mine(m)) continue;
    Vec<TO, V> o;
#pragma unroll
    for (int q = 0; q < V; ++q) o.v[q] = TO(sv[m][q] + (GA[at_a(m) + q] + GB[at_b(m) + q * rs]));
    *reinterpret_cast<Vec<TO, V> *>(reinterpret_cast<char *>(Oe) +
                                    (uint32_t)(V * (lane + 64 * m)) * (uint32_t)sizeof(TO)) = o;
  }
}

// ---------------------------------------------------------------------------
// k_hwave (Hermite basis, two and three modes): a whole RK4 stage of one q cube
// ---------------------------------------------------------------------------
// Same task, task order, inputs and result as k_hcube, in the wave-plane form:
// a task is one (branch, element, Hermite index k) and its block the q grid.
// Three modes (MM = 3): planes (q_2, q_3) over q_1, as k_pwave; the RK4 stage
// update is applied as each wave stores.  Two modes (MM = 2): the block is
// one (q_1, q_2) plane, a wave takes a task by itself and no barrier is left
// (k_hcube gave each task one workgroup with a lane per q_2 point).
// A missing neighbour is the task's own block with zero factors (an L1 hit).
// Per stage, before and after: 24^3 x 12^3 FP64 4.9 -> 2.5 ms, four FP32
// states 12.4 -> 6.9 ms; 32^2 x 16^2 FP64 0.140 -> 0.024 ms.  At 24^3 it is
// bound by the reads that miss L2 (FP64: 8.1 states a launch, 6.9 TB/s with the
// writes; its twelve neighbour blocks and the force tables).  The task order
// set for k_hcube is its best too: chunks of 10 to 240 tasks and k_2 tiles of 2
// to 6 move it by -0.5 to +6%, one range per XCD by +18%.
constexpr int hwave_npw(const int nb, const bool exact, const int mm) { return mm == 2 ? 1 : pwave_npw(nb, exact); }
constexpr int hwave_ps(const int nb, const bool exact, const int mm) { return mm == 2 ? 1 : wave_ps(nb, exact); }
constexpr int hwave_waves(const int nb, const bool exact, const int mm) {
  return mm == 2 ? 4 : pwave_waves(nb, exact);
}
constexpr size_t hwave_lds_vals(const int nb, const int n1, const int n2, const int n3, const int nw, const int ps,
                                const int mm) {
  return (mm == 2 ? 2 * (size_t)nw * (wave_slot(n2, n3, 1) + 16)
                  : (size_t)(n1 + nw * ps) * wave_slot(n2, n3, ps) + wave_pad(nb, ps)) +
         (mm == 2 ? 2 * (size_t)nw : 3) * (size_t)nb;
}
constexpr int hwave_occ(const int nb, const int tsize) { return nb >= 24 ? 2 : tsize == 4 ? 4 : 3; }

// epi: the stage update (an Epi; uniform, so one kernel serves all stages).
template <typename T, int NB, int NVR, int MM>
__global__ void __launch_bounds__((64 * hwave_waves(NB, NVR == 0, MM)), (hwave_occ(NB, sizeof(T))))
k_hwave(const Geom g, const Tabs tb, const PCube pc, const T *__restrict__ X, const T *__restrict__ y,
        T *__restrict__ out, const double cst, const int epi) {
  constexpr bool EXACT = NVR == 0;
  constexpr int V = wave_vec(sizeof(T), EXACT);
  constexpr int PS = hwave_ps(NB, EXACT, MM);
  constexpr int NV = EXACT ? wave_nv(NB, PS, V) : NVR;
  constexpr int NPW = hwave_npw(NB, EXACT, MM);
  constexpr int A2 = MM - 2, A3 = MM - 1;  // modes of the rows and columns of a plane
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nw = EXACT ? hwave_waves(NB, EXACT, MM) : (int)(blockDim.x >> 6);
  const int wg = pc.chunk > 0 ? xcd_chunk_task(blockIdx.x, pc.chunk) : xcd_task(blockIdx.x, pc.nblk);
  // two modes: a workgroup's waves take consecutive tasks (waves past the last task redo it and store nothing)
  if ((MM == 2 ? wg * nw : wg) >= pc.ntasks) return;
  const int task = MM == 2 ? min(wg * nw + w, pc.ntasks - 1) : wg;
  const int N1 = EXACT ? (MM == 2 ? 1 : NB) : pc.N1, N2 = EXACT ? NB : pc.N2, N3 = EXACT ? NB : pc.N3;
  const int plane = EXACT ? NB * NB : pc.plane;
  const int rs = wave_rs(N2, N3);
  const int slot = wave_slot(N2, N3, PS);
  T *tiles = reinterpret_cast<T *>(smem_raw);
  T *own = tiles + (MM == 2 ? nw * (slot + 16) : N1 * slot + wave_pad(NB, PS));
  // V' by mode; two modes: a copy per wave (V1 stays unused)
  T *V1 = own + (MM == 2 ? nw * (slot + 16) : nw * PS * slot);
  T *V2 = MM == 2 ? V1 + 2 * w * NB : V1 + NB, *V3 = V2 + NB;
  const int per_br = g.ne * g.P;
  const int br = task / per_br;
  const int kb = (task - br * per_br) / g.ne;
  const int e = task - br * per_br - kb * g.ne;  // the elements of one k are adjacent tasks
  const int kl = hcube_kl(g, pc.ktile, kb);      // Hermite multi-index, k_M fastest in storage
  const long long Q = g.Q;
  const long long slice = ((long long)(br * g.ne + e) * g.P + kl) * Q;  // this task's q block
  const T *Xe = X + slice;
  const T *Xb = X + (long long)br * g.ne * g.E;  // this branch's element 0
  // c_{k+e}, c_{k-e}, c_{n+e,k-e}, c_{n-e,k+e} and their factors: in the q
  // derivative's field (GU, GD, times cb: see wave_rhs), the force term (FU,
  // FD) and the couplings (PH, TH)
  const T *Xu[MM], *Xd[MM], *Hu[MM], *Hd[MM];
  T GU[MM], GD[MM], FU[MM], FD[MM], PH[MM], TH[MM];
  bool any_up = false;
  {
    int rem = kl;
#pragma unroll
    for (int s = MM - 1; s >= 0; --s) {
      const int ks = rem % g.Np[s];
      rem /= g.Np[s];
      const bool kup = ks + 1 < g.Np[s], kdn = ks > 0;
      const int up = tb.up[e * 3 + s], dn = tb.dn[e * 3 + s];
      any_up = any_up || up >= 0;
      const long long st = (long long)g.PS[s] * Q;
      Xu[s] = kup ? Xe + st : Xe;
      Xd[s] = kdn ? Xe - st : Xe;
      Hu[s] = (kdn && up >= 0) ? Xb + ((long long)up * g.P + kl) * Q - st : Xe;
      Hd[s] = (kup && dn >= 0) ? Xb + ((long long)dn * g.P + kl) * Q + st : Xe;
      const double sp = kup ? sqrt((double)(ks + 1)) : 0.0;  // zero past the truncation
      const double sm = kdn ? sqrt((double)ks) : 0.0;
      GU[s] = uniform(T(-g.ha[s] * sp * g.dq_cb[s]));
      GD[s] = uniform(T(-g.ha[s] * sm * g.dq_cb[s]));
      FU[s] = uniform(T(g.hf[s] * sp));
      FD[s] = uniform(T(-g.hf[s] * sm));
      PH[s] = uniform(T(up >= 0 ? -g.hl[s] * sm : 0.0));
      TH[s] = uniform(T(tb.cc[e * 3 + s] * g.hl[s] * sp));  // cc is zero when n_s = 0
    }
  }
  const T dmp = uniform(T(tb.damp[e]));
  // The V' tables come to LDS behind the first loads of the planes.  Three modes:
  // the workgroup has one task, one element, and meets at a barrier.  Two modes:
  // the waves branch apart on their elements below, so each keeps its own copy
  // and waits for nobody.
  const int ti = MM == 2 ? lane : tid, tl = min(ti, NB - 1);
  const T tv1 = MM == 3 ? T(tb.Vp[tl]) : T(0), tv2 = T(tb.Vp[A2 * kTab + tl]), tv3 = T(tb.Vp[A3 * kTab + tl]);
  auto fill_tables = [&]() {
    if (ti < NB) {
      if constexpr (MM == 3) V1[ti] = tv1;
      V2[ti] = tv2;
      V3[ti] = tv3;
    }
    if constexpr (MM == 3)
      __syncthreads();
    else
      wave_lds_fence();
  };

  // vectors of this lane (as in k_pwave)
  constexpr int PER0 = NB / V / wave_gcd(NB / V, 64);
  constexpr int DR = 64 * V * PER0 / NB;
  constexpr bool REP = EXACT && PER0 < NV && PS == 1;
  constexpr int PER = REP ? PER0 : NV;
  int row[PER], col[PER], pln[PER];
#pragma unroll
  for (int m = 0; m < PER; ++m) {
    const int idx = min(V * (lane + 64 * m), PS * plane - V);
    pln[m] = PS > 1 ? idx / plane : 0;
    const int in = idx - pln[m] * plane;
    row[m] = in / N3;
    col[m] = in - row[m] * N3;
  }
  auto at_a = [&](const int m) { return pln[m % PER] * slot + row[m % PER] * rs + col[m % PER] + m / PER * (DR * rs); };
  auto at_b = [&](const int m) { return pln[m % PER] * slot + col[m % PER] * rs + row[m % PER] + m / PER * DR; };
  auto mine = [&](const int m) {
    return (EXACT && V * 64 * (m + 1) <= PS * NB * NB) || V * (lane + 64 * m) < PS * plane;
  };
  // first point of vector m of group k, within the block (lanes past a plane re-read its last vector)
  auto point = [&](const int k, const int m) {
    uint32_t o = (uint32_t)((w + k * nw) * (MM == 2 ? 0 : PS * plane));
    asm volatile("" : "+s"(o));  // keeps the loads where they are issued (see k_pwave)
    const uint32_t at = (uint32_t)(V * (lane + 64 * m));
    return o + (EXACT && V * 64 * (m + 1) <= PS * NB * NB ? at : min(at, (uint32_t)(PS * plane - V)));
  };
  auto get = [&](const auto *p, const uint32_t at) {
    using E = std::remove_const_t<std::remove_pointer_t<decltype(p)>>;
    return *reinterpret_cast<const Vec<E, V> *>(reinterpret_cast<const char *>(p) + at * (uint32_t)sizeof(E));
  };

  struct In {
    Vec<T, V> c, u[MM], d[MM], a[MM], b[MM];
    Vec<double, V> F[MM];
  };
  T sv[NPW][NV][V];
  auto sweep = [&](auto UP) {
    constexpr bool up = decltype(UP)::value;
    auto load = [&](const int k, const int m) {
      In x;
      const uint32_t at = point(k, m);
      x.c = get(Xe, at);
#pragma unroll
      for (int s = 0; s < MM; ++s) {
        x.u[s] = get(Xu[s], at);
        x.d[s] = get(Xd[s], at);
        if constexpr (up) x.a[s] = get(Hu[s], at);
        x.b[s] = get(Hd[s], at);
        x.F[s] = get(tb.F + s * Q, at);
      }
      return x;
    };
    In nxt = load(0, 0);
    fill_tables();
#pragma unroll
    for (int k = 0; k < NPW; ++k) {
      const int i0 = MM == 2 ? 0 : (w + k * nw) * PS;
      if (!EXACT && i0 >= N1) break;  // uniform over the wave
      Vec<T, V> g1[NV];
      T *GA = MM == 2 ? tiles + w * (slot + 16) : tiles + i0 * slot;
      T *GB = MM == 2 ? own + w * (slot + 16) : own + w * PS * slot;
#pragma unroll
      for (int m = 0; m < NV; ++m) {
        const In x = nxt;
        const T v2 = V2[row[m % PER] + m / PER * DR];
        const T v1 = MM == 3 ? V1[i0 + pln[m % PER]] : T(0);
        Vec<T, V> f2, f3;
#pragma unroll
        for (int q = 0; q < V; ++q) {
          T s = -dmp * x.c.v[q];
#pragma unroll
          for (int a = 0; a < MM; ++a) {
            const T u = x.u[a].v[q], d = x.d[a].v[q];
            s += T(x.F[a].v[q]) * (FU[a] * u + FD[a] * d);
            T t = TH[a] * x.b[a].v[q];
            if constexpr (up) t += PH[a] * x.a[a].v[q];
            s += (a == A3 ? V3[col[m % PER] + q] : a == A2 ? v2 : v1) * t;
          }
          f2.v[q] = GU[A2] * x.u[A2].v[q] + GD[A2] * x.d[A2].v[q];
          f3.v[q] = GU[A3] * x.u[A3].v[q] + GD[A3] * x.d[A3].v[q];
          if constexpr (MM == 3) {
            T a1 = GU[0] * x.u[0].v[q] + GD[0] * x.d[0].v[q];
            asm volatile("" : "+v"(a1));
            g1[m].v[q] = a1;
          }
          asm volatile("" : "+v"(s));  // formed here: its inputs are not kept
          sv[k][m][q] = s;
        }
        if (m + 1 < NV)
          nxt = load(k, m + 1);
        else if (k + 1 < NPW && (EXACT || i0 + nw * PS < N1))
          nxt = load(k + 1, 0);
        if (mine(m)) {
#pragma unroll
          for (int q = 0; q < V; ++q) GA[at_a(m) + q] = f2.v[q];
#pragma unroll
          for (int q = 0; q < V; ++q) GB[at_b(m) + q * rs] = f3.v[q];
        }
      }
      wave_lds_fence();
      plane_solve<T, NB, PS, EXACT, false>(GA, GB, lane, N2, N3, rs, slot, nullptr, nullptr);
      wave_lds_fence();
#pragma unroll
      for (int m = 0; m < NV; ++m) {
        if (!mine(m)) continue;
#pragma unroll
        for (int q = 0; q < V; ++q) sv[k][m][q] += GA[at_a(m) + q] + GB[at_b(m) + q * rs];
      }
      if constexpr (MM == 3) {
        wave_lds_fence();
#pragma unroll
        for (int m = 0; m < NV; ++m) {
          if (!mine(m)) continue;
#pragma unroll
          for (int q = 0; q < V; ++q) GA[at_a(m) + q] = g1[m].v[q];
        }
      }
    }
  };
  if (any_up)  // the elements below the hierarchy's last level; uniform over a task
    sweep(std::true_type{});
  else
    sweep(std::false_type{});
  if constexpr (MM == 3) {
    __syncthreads();
    // q_1 lines, one per thread, in place in the tiles
    for (int l = tid; l < plane; l += blockDim.x) {
      const int r2 = l / N3;
      wave_line<T, NB, EXACT, false>(tiles + r2 * rs + (l - r2 * N3), slot, N1, true, nullptr);
    }
    __syncthreads();
  }
  if (MM == 2 && wg * nw + w >= pc.ntasks) return;
  T *Oe = out + slice;
  // what the stage update adds to: out = base + cst x (EPI_OUT: the right-hand side x itself)
  const T *Be = epi == EPI_H1 ? Xe : epi == EPI_H2 ? y + slice : Oe;
  const T cs = epi == EPI_OUT ? T(1) : T(cst);
#pragma unroll
  for (int k = 0; k < NPW; ++k) {
    const int i0 = MM == 2 ? 0 : (w + k * nw) * PS;
    if (!EXACT && i0 >= N1) break;
    Vec<T, V> base[NV];
    if (epi != EPI_OUT) {
#pragma unroll
      for (int m = 0; m < NV; ++m) base[m] = get(Be, point(k, m));
    } else {
#pragma unroll
      for (int m = 0; m < NV; ++m) base[m] = Vec<T, V>{};
    }
#pragma unroll
    for (int m = 0; m < NV; ++m) {
      if (!mine(m)) continue;
      Vec<T, V> o;
#pragma unroll
      for (int q = 0; q < V; ++q) {
        T x = sv[k][m][q];
        if constexpr (MM == 3) x += tiles[i0 * slot + at_a(m) + q];
        o.v[q] = base[m].v[q] + cs * x;
      }
      *reinterpret_cast<Vec<T, V> *>(reinterpret_cast<char *>(Oe) +
                                     (uint32_t)(i0 * plane + V * (lane + 64 * m)) * (uint32_t)sizeof(T)) = o;
    }
  }
}

}  // namespace chfpe
