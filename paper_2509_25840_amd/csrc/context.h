// State of a solver context and the launch plan, shared by the host side
// (chfpe.hip) and the launchers of the kernel families (launch_*.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>
#include <string>
#include <type_traits>
#include <vector>

#include "chfpe.h"
#include "kernels.h"
#include "one.h"
#include "qcube.h"
#include "staging.h"
#include "wave.h"

namespace chfpe {

constexpr int kPBlockRPT = 4;        // rows per k_pblock thread
constexpr int kNumBase = 15;         // kernel kinds of the event timing (see Kind in chfpe.hip)
constexpr int kNumKinds = 2 * kNumBase + 2;

struct Derived {
  int prec = 0, B = 1;    // precision of branch states; branches per wave
  bool batched = false;   // 2D responses use the batched branch buffers
  bool hermite = false;   // Hermite basis in p: P counts Hermite functions, layout [n][k][q]
  int M = 0, K = 0, ne = 0;
  int Nq[3] = {0, 0, 0}, Np[3] = {0, 0, 0};  // axes s >= M stay 0
  int Q = 0, P = 0;
  long long E, S;  // points per element, values per state
  std::vector<int> nvec;  // ne * M
};

inline int nmax_bucket(int n) {
  return n <= 8 ? 8 : n <= 12 ? 12 : n <= 16 ? 16 : n <= 24 ? 24 : n <= 32 ? 32 : 48;
}

inline int pcube_n3(const Derived &d) { return d.M == 3 ? d.Np[2] : 1; }

constexpr int kStateBufs = 6;   // FP64: W_eq, U, y, xa, xb, t
constexpr int kBranchBufs = 4;  // per branch of a wave: y, xa, xb, t

// Workspace layout (byte offsets, 256-aligned).
struct Layout {
  size_t F, VpQ, Vp, pm, pg, gA, gB, gC, Cw, wp, sq, sp, up, dn, cc, tc, damp, partial, scal, flag, clos;
  size_t bufs[kStateBufs];
  size_t bbufs[kBranchBufs];  // batched branch buffers: y, xa, xb, t (B states each)
  size_t total;
};
struct Launch {
  PBlock pb{};
  size_t pb_lds = 0;
  int pb_threads = 256, pb_nmax = 48;
  int pb_rpt = 4;  // rows per k_pblock thread (3 where it tiles the 24-row blocks exactly)
  // strided-axis passes of one stage: qa (three modes only, accumulates into
  // t) then qf (applies the stage update); qx: the p_1 excitation pass of
  // three modes.
  QPass qa{}, qf{}, qx{};
  bool has_qa = false, qf_two = false, has_qx = false;
  // three modes: all p axes of a q point in one k_pcube task (then the q
  // passes are (q_2, q_3) and q_1 alone, and excitations need no qx)
  bool pcube = false, pcube_split = false;
  bool pcube_s = false;  // k_pcube_s rather than k_pcube
  bool pwave = false;    // k_pwave can take the block (p axes of at most 24 points), where it pays
  int pwave_nb = 0;
  // two modes: the p side by k_pwave2 (p axes of at most 32 points)
  bool pwave2 = false;
  int pwave2_nb = 0;
  PCube pw2{};
  PCube pcb{};
  // three modes: every q derivative and the stage update in one pass (k_qcube)
  bool qcube = false;
  // Hermite basis: k_hcube over the q cube of each (branch, element, k)
  bool hcube = false;
  PCube hcb{};
  int hcube_threads = 0, hcube_nb1 = 0;
  bool hwave = false;  // k_hwave can take it (three modes, q axes of at most 24 points; two modes, 32)
  int hwave_nb = 0;
  int pcube_threads = 0, pcube_nb1 = 0;
  // one mode: whole propagations by one workgroup per state (k_one)
  bool one = false;
  int qa_threads = 0, qf_threads = 0, qx_threads = 0;
  size_t qa_lds = 0, qf_lds = 0;
  int qa_nmax = 48, qf_nmax = 48, qx_nmax = 48;
};

inline int pad8(int n) { return (n + 7) / 8 * 8; }
// k_hcube grid: a multiple of 8 chunks when the tasks go to the XCDs in chunks
inline int hcube_nblk(int ntasks, int chunk) { return chunk > 0 ? (ntasks + 8 * chunk - 1) / (8 * chunk) * (8 * chunk) : pad8(ntasks); }

// k_pwave2 grid: a wave per task
inline int pwave2_nblk(int ntasks) { return pad8((ntasks + kPWave2Waves - 1) / kPWave2Waves); }

}  // namespace chfpe

using namespace chfpe;

struct chfpe_ctx {
  chfpe_params prm;
  Derived d;
  Layout L;
  Launch ln;
  Geom g;
  Tabs tb;
  hipStream_t stream = nullptr;
  unsigned char *ws = nullptr;
  bool own_ws = false;
  double *F, *VpQ, *Vp, *pm, *pg, *gA, *gB, *gC, *Cw, *wp, *sq, *sp, *cc, *tc, *damp, *partial, *scal;
  int *up, *dn, *flag;
  double *weq, *u, *y, *xa, *xb, *t;
  void *bb[kBranchBufs] = {nullptr, nullptr, nullptr, nullptr};  // batched y, xa, xb, t
  // cached graph of one wave's t2 loop
  hipGraphExec_t wave_graph = nullptr;
  long long wave_key[6] = {0, 0, 0, 0, 0, 0};
  bool has_eq = false;
  double dV = 1.0;
  std::vector<double> qgrid[3], pgrid[3];
  std::vector<double> wq_host;  // q-point weights (product over q axes), Q entries
  std::vector<double> sq_host;  // exp(-beta U(q)/2), Q entries
  Staging staging;  // host copies of whole states
  double *rbuf = nullptr;
  size_t rbuf_cap = 0;
  std::string err = "no error";
  int tune_pb_nb = 0;   // blocks per k_pblock task (0: automatic)
  int tune_q_pc = 0;    // run positions per two-axis k_qpass tile (0: automatic)
  int tune_pb_split = -1;  // k_pblock lines solved by lane pairs (-1: automatic)
  int tune_pb_run = 0;     // k_pblock consecutive block groups per state in task order (0: 1)
  int tune_pc_pad = 0;     // k_pcube LDS plane row pad (0: 1)
  int tune_pc_stream = -1;  // k_pcube_s (1) or k_pcube (0); -1: by the p_1 length
  int tune_hc_chunk = -1;   // k_hcube tasks per XCD chunk (0: one contiguous range per XCD; -1: automatic)
  int tune_hc_ktile = 0;    // k_hcube k_2 tile of the task order (0: automatic)
  bool capturing = false;  // a HIP graph is being captured: no event timing
  bool closure_on = false; // right-hand sides use the closure stencil weights (tb.clos)
  bool use_graphs = true;
  bool allow_pcube = true;  // three modes: k_pcube where the p block fits it
  bool allow_pwave = true;  // three modes: k_pwave where a wave's lines hold the p axes
  bool allow_hwave = true;  // Hermite basis: k_hwave where a wave's lines hold the q axes
  bool allow_pwave2 = true; // two modes: k_pwave2 where a wave's lines hold the p axes
  bool allow_qcube = true;  // three modes: k_qcube where the q cube fits it
  bool allow_one = true;    // one mode: k_one where the state fits it
  // kernel timing
  int timing_every = 0;
  long long step_counter = 0;
  bool timing_now = false;
  struct Pending {
    hipEvent_t a, b;
    int kind;
    double bytes;
  };
  std::vector<Pending> pending;
  std::vector<hipEvent_t> event_pool;
  long long kcount[kNumKinds] = {0};
  double ktime[kNumKinds] = {0};
  double kbytes[kNumKinds] = {0};
};

namespace chfpe {

// LDS of a k_pcube workgroup: a copy of the task's p block, and two fields
// of one round's (p_2, p_3) planes with rows of N_3 + pad values.  The
// streamed form (k_pcube_s) keeps no copy: its planes, and the first
// forward results of every p_1 line.
inline size_t pcube_lds_bytes(const Derived &d, size_t tsize, int pad, bool stream) {
  const int nb1 = nmax_bucket(d.Np[0]);
  const size_t rows = (size_t)d.Np[1] * (size_t)(pcube_n3(d) + pad);
  if (stream)
    return (kPCubeCF + 2 * (size_t)pcube_s_planes(nb1) * rows +
            (size_t)pcube_s_dlds((int)tsize, nb1) * d.Np[1] * pcube_n3(d)) * tsize;
  return ((size_t)d.P + 2 * (size_t)pcube_planes(nb1) * rows + (size_t)d.Np[0]) * tsize;  // + the p_1 table
}

// LDS values of a k_one workgroup.
inline size_t one_lds_vals(const Derived &d) {
  // (the reads ahead of a line may run past the last array, into the tables)
  static_assert(kStreamPF * one_rs(kMaxAxis) <= kOneTables, "reads ahead stay in the allocation");
  const int n = std::max(d.Nq[0], d.Np[0]);
  return (size_t)2 * d.ne * n * one_rs(one_bucket(n)) + kOneTables;
}
// k_one takes the one-mode grids that fit its registers and LDS.
inline bool one_shape_ok(const Derived &d) {
  return d.M == 1 && !d.hermite && d.ne <= kOneMaxElements &&
         one_fits(sizeof(double), one_bucket(std::max(d.Nq[0], d.Np[0])), one_ne(d.ne));
}

// Waves of a k_pwave workgroup.
inline int pwave_nw(const PCube &p, int nb) {
  const bool exact = p.N1 == nb && p.N2 == nb && p.N3 == nb;
  const int per = wave_ps(nb, exact) * pwave_npw(nb, exact);
  return (p.N1 + per - 1) / per;
}

// Where k_pwave is the faster form of a block of n1 planes of `plane` points,
// lines in the nb bucket; below, k_pcube (p_1 axes up to 16 points and no
// closure: k_pcube_s).  A wave goes through its planes one by one, with all nb
// steps of a line solve and all vectors of its variant however few lines and
// points they have, and n1 sets how many workgroups share a CU's eight waves
// (24-point lines, 13 to 16 planes: one of five or six waves); k_pcube's cost
// follows the points in waves of 64.  RK4 steps at 504 q points and four elements,
// k_pcube[_s] and k_pwave, FP64 and four FP32 states, in us:
//   24 x 5 x 5    226  506,  392  757    24 x 12 x 12  717  747, 1701 1335
//   24 x 9 x 18   781  777, 1816 1436    24 x 16 x 16 1112  986, 2461 2031
//   17 x 13 x 17  711  756, 1814 1516    17 x 10 x 24  788  780, 1968 1576
//   16 x 8 x 17   415  571,  809 1114    16 x 15 x 17  605  731, 1417 1533
//   16 x 16 x 17  941  822, 1972 2194    10 x 10 x 17  343  376,  678  651
//   8 x 15 x 17   388  424,  847  682    8 x 16 x 17   566  460, 1277  795
//   5 x 6 x 18    157  195,  303  300    5 x 8 x 17    221  225,  402  345
//   16 x 8 x 8    223  233,  370  420    16 x 9 x 9    254  262,  500  489
//   16 x 10 x 10  282  287,  565  534    13 x 11 x 11  277  275,  563  514
//   12 x 8 x 8    196  200,  315  343    12 x 9 x 9    210  220,  418  394
//   8 x 7 x 9     157  149,  250  240    8 x 5 x 5     123  103,  182  146
//   5 x 5 x 9     114  116,  169  178    5 x 7 x 9     127  122,  191  189
// and with a closure 16 x 8 x 8 269 298, 16 x 9 x 9 380 329, 12 x 10 x 10 269
// 281, 9 x 7 x 13 227 245, 5 x 11 x 13 287 237.
inline bool pwave_pays(int nb, int n1, int plane, size_t tsize, bool clos) {
  if (nb <= 8) return true;
  if (clos) return plane > (nb == 16 && n1 > 12 ? 64 : 100);
  if (nb <= 16) return plane > (n1 <= 8 ? 48 : tsize == 4 ? 64 : nb <= 12 ? 110 : 90);
  if (tsize == 4) return plane > (n1 <= 6 ? 96 : n1 > 12 && n1 <= 16 ? 400 : 128);
  return plane > (n1 <= 6 ? 128 : n1 <= 16 ? 256 : n1 < 24 ? 224 : 150);
}
// The same for three-mode k_hwave and k_hcube, by the q cube: steps of 4 x 5 x 4
// functions and ten elements, k_hcube and k_hwave, FP64 and four FP32 states:
//   24 x 5 x 5    214  410,  249  746    24 x 13 x 13  328  445,  869  860
//   24 x 11 x 18  625  448,  934  890    17 x 14 x 14  467  384,  707  840
//   17 x 15 x 17  488  385,  736  859    17 x 16 x 17  973  404, 1361  899
//   16 x 8 x 17   227  345,  429  722    16 x 15 x 17  276  365,  646  804
//   12 x 10 x 20  204  229,  479  349    12 x 8 x 20   193  222,  356  334
//   10 x 9 x 18   159  207,  294  319    5 x 13 x 20   276  124,  358  224
//   5 x 8 x 20    104  111,  188  199    16 x 7 x 7    174  172,  203  236
//   13 x 8 x 8    161  167,  185  220    16 x 9 x 9    190  179,  339  248
//   12 x 5 x 5    115   99,  137  155    12 x 8 x 8    145  102,  169  163
inline bool hwave_pays(int nb, int n1, int plane, size_t tsize) {
  if (nb <= 8) return true;
  if (tsize == 8) return plane > (nb <= 12 ? 0 : nb <= 16 ? (n1 < 16 ? 64 : 48) : n1 > 16 ? 192 : 256);
  if (nb <= 16) return plane > (nb <= 12 ? 63 : 64);
  return plane > (n1 <= 10 ? 192 : n1 <= 12 || n1 == 24 ? 136 : 256);
}
// Where k_pwave2 is the faster form for a launch of `tasks` planes: a task is a
// wave however small its plane, and once there are several waves for every slot
// of the device k_pblock packs small planes better.  RK4 steps of 20 x 24 q
// points and six elements, k_pblock and k_pwave2, FP64: 25 x 5 points, one state
// 88 79 us, 8 states 189 232, 32 states 716 904; 32 x 5, 1 and 16 states 96 83,
// 451 507; 32 x 6, 99 86, 515 558; 25 x 8, 97 87, 565 550; 20 x 5, 82 73, 285
// 307; 24 x 6, 88 76, 394 354; 8 x 8, 8 and 32 states 105 115, 229 288; 9 x 5, 1
// and 16 states 70 62, 166 185 (FP32 142 151); 5 x 5, 70 61, 180 169 (148 134);
// 13 x 5, 76 69, 248 233.  Larger planes of FP32 gain.
inline bool pwave2_pays(int nb, int plane, size_t tsize, long long tasks) {
  if (nb <= 12) return plane <= 32 || plane > 64 || tasks <= 16384;
  if (nb <= 16 || tsize == 4) return true;
  return plane > (nb <= 24 ? 120 : 196) || tasks <= 8192;
}

// Waves of a k_hwave workgroup, and its workgroups for ntasks tasks (two
// modes: a wave per task).
inline int hwave_nw(const Derived &d, const PCube &p, int nb) {
  const bool exact = (d.M == 2 || p.N1 == nb) && p.N2 == nb && p.N3 == nb;
  if (d.M == 2) return hwave_waves(nb, exact, 2);
  const int per = hwave_ps(nb, exact, 3) * hwave_npw(nb, exact, 3);
  return (p.N1 + per - 1) / per;
}

template <typename K>
void allow_lds(K kern, size_t bytes) {
  if (bytes > 64 * 1024)
    (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

// A launch description for nb states stored back to back (t1 branches).
struct Batch {
  Geom g;
  PBlock pb;
  PCube pcb, pw2, hcb;
  QPass qa, qf, qx;
};

// Closure variants of the kernels exist for FP64 states with every axis in a
// bucket of at most 16 points (chfpe_set_closure enforces this).
template <typename T, typename TO, int NMAX>
constexpr bool kClosureBuilt = std::is_same<T, double>::value && std::is_same<TO, double>::value && NMAX <= 16;

}  // namespace chfpe
