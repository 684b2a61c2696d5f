// Device code of the vertex-patch smoother that more than one source file's kernels run: tables, 1D products,
// the eigenbasis and additive passes with their launch shapes.
#pragma once
#include "device_common.hpp"
#include "kernels.hpp"
#include "patch_tables_gen.hpp"

#include <cmath>
#include <type_traits>
#include <vector>

namespace vps {

// The including file's own copy, filled by upload_tables().
static __constant__ DevTables<double> g_tab64[kMaxDegree + 1];
static __constant__ DevTables<float> g_tab32[kMaxDegree + 1];

template <typename T>
__device__ __forceinline__ const DevTables<T>& tab(int k);
template <>
__device__ __forceinline__ const DevTables<double>& tab<double>(int k) { return g_tab64[k]; }
template <>
__device__ __forceinline__ const DevTables<float>& tab<float>(int k) { return g_tab32[k]; }

// Launch shape per (dim, degree): patches per workgroup and threads.
template <int D, int K>
struct SmootherShape;
// Degrees (bit K) whose 2D shape takes one wave (64 threads, half the patches) instead of two:
// measured 1-3% faster per V-cycle at degrees 3, 4, 5 and 7, equal at 2 and 6, slower at 1.
#ifndef VPS_2D_WAVE_MASK
#define VPS_2D_WAVE_MASK 0xB8
#endif
template <int K> struct SmootherShape<2, K> {
  static constexpr bool ONE_WAVE = ((VPS_2D_WAVE_MASK) >> K) & 1;
  static constexpr int PPW = (K == 1 ? 64 : K == 2 ? 32 : K == 3 ? 16 : K <= 5 ? 12 : 8) / (ONE_WAVE ? 2 : 1);
  static constexpr int NT = ONE_WAVE ? 64 : 128;
};
template <int K> struct SmootherShape<3, K> {
  static constexpr int PPW = K == 1 ? 32 : K == 2 ? 8 : K == 3 ? 4 : K == 4 ? 2 : 1;
  static constexpr int NT = K <= 5 ? 128 : K == 6 ? 192 : 256;
  // the default shape of the residual form shares one LDS region between the closure and the
  // first two contraction stages (see SmootherLds): measured 2-13% faster for degrees 3-7 (occupancy),
  // no gain for degrees 1-2, where the layout is already small
  static constexpr bool ALIAS = K >= 3;
};

// Patches per workgroup for small launches (coarse levels): fewer patches per workgroup means
// fewer tasks per thread in every stage, so a workgroup finishes sooner; used when the default
// shape would give fewer than kLatencyBlocks workgroups, where the chip is not full anyway.
template <int D, int K>
struct LatencyPPW {
  static constexpr int value = D == 3 ? (K == 1 ? 8 : K == 2 ? 2 : 1) : (K == 1 ? 16 : K == 2 ? 8 : K <= 5 ? 4 : 2);
};
#ifndef VPS_LATENCY_BLOCKS
#define VPS_LATENCY_BLOCKS 1024
#endif
constexpr long long kLatencyBlocks = VPS_LATENCY_BLOCKS;

// Two words of T moved by one 8- or 16-byte LDS access.
template <typename T>
struct Pair;
template <>
struct Pair<float> {
  using type = float2;
};
template <>
struct Pair<double> {
  using type = double2;
};

// Smallest s >= v with s = r (mod 32): padded outer strides of the LDS transpose buffers.
constexpr int pad32(int v, int r) { return v + ((r - v) % 32 + 32) % 32; }

// LDS layouts.  Every transpose buffer puts the loop axis of the stage that reads it outermost,
// so the reading lanes touch consecutive words; the outer stride is padded (mod 32) so that the
// writing lanes of the previous stage also fall into distinct banks.
template <int D, int K, typename T, int PPWv, bool ALIASv = false, bool PAIRv = false>
struct SmootherLds {
  static constexpr int n = 2 * K + 1, m = 2 * K - 1;
  static constexpr int PPW = PPWv;
  static constexpr int RS = 2 * K * PPW + 1;  // closure row segment of the workgroup
  // ---- 3D strides
  // residue of the P stride that makes the x0-contraction writes conflict-free (searched per degree
  // for the launch shapes above, 4- and 8-byte words)
  static constexpr int kSJ1Res[8] = {0, 11, 7, 19, 15, 27, 23, 3};
  static constexpr int SJ1 = pad32(PPW * n * m, kSJ1Res[K]);  // P  [j1][q][j2][i0]   (PM, PA)
  static constexpr int SJ2 = pad32(PPW * m * m, m);          // UV [j2][q][i1][i0]   (U, V)
  static constexpr int SI1 = pad32(PPW * m * m, m);          // W4 [i1][q][a2][i0]
  static constexpr int SI0 = pad32(PPW * m * m, 1);          // W5 [i0][q][a2][a1]
  static constexpr int SA1 = pad32(PPW * m * m, 1);          // W6 [a1][q][a2][i0]
  static constexpr int SA2 = pad32(PPW * m * m, m);          // W7 [a2][q][i1][i0]
  static constexpr int X3 = n * n * RS;
  static constexpr int P3 = 2 * n * SJ1;
  static constexpr int UV3 = 2 * n * SJ2;
  static constexpr int A3 = P3 > m * SI1 ? (P3 > m * SA1 ? P3 : m * SA1) : (m * SI1 > m * SA1 ? m * SI1 : m * SA1);
  static constexpr int B3a = X3 > UV3 ? X3 : UV3;
  static constexpr int B3b = m * SI0 > m * SA2 ? m * SI0 : m * SA2;
  static constexpr int B3 = B3a > B3b ? B3a : B3b;
  // ---- 2D strides
  static constexpr int T1 = pad32(PPW * m, (m * PPW) % 32);  // P2  [j1][q][i0]  (PM, PA)
  static constexpr int T0 = pad32(PPW * m, 1);               // W   [i0][q][a1]
  static constexpr int TA = pad32(PPW * m, 1);               // W2  [a1][q][i0]
  static constexpr int X2 = n * RS;
  static constexpr int P2 = 2 * n * T1;
  static constexpr int A2 = P2 > m * TA ? P2 : m * TA;
  static constexpr int B2 = X2 > m * T0 ? X2 : m * T0;
  // ---- aliased 3D layout (multiplicative): the closure X, PM/PA and U/V all start at word 0 (the x0
  // and x1 stages read their inputs into registers and the workgroup synchronises before they
  // write), the x2 and x0 diagonalisation outputs (W4, W6) follow U/V, the x1 ones (W5, W7) start
  // at 0 again once U/V is dead
  static constexpr bool AL = ALIASv && D == 3;
  static constexpr int W46 = m * SI1 > m * SA1 ? m * SI1 : m * SA1;
  static constexpr int W57 = m * SI0 > m * SA2 ? m * SI0 : m * SA2;
  static constexpr int AL3a = X3 > P3 ? X3 : P3;
  static constexpr int AL3 = AL3a > UV3 + W46 ? AL3a : UV3 + W46;
  // ---- paired 3D layout (aliased, smaller still): PM and PA interleaved as pairs [j1][q][j2][i0]{M, A}
  // (one 8-byte access per pair, the pair stride SJP padded for conflict-free writes of the x0
  // stage), W4 also over U/V (the x2 stage synchronises before it writes), W5 and W7 after W4/W6
  static constexpr bool PR = PAIRv && AL;
  static constexpr int SJP = pad32(2 * PPW * n * m, 30);
  static constexpr int PP3 = n * SJP;
  static constexpr int PR3a = X3 > PP3 ? X3 : PP3;
  static constexpr int PR3b = UV3 > W46 + W57 ? UV3 : W46 + W57;
  static constexpr int PR3 = PR3a > PR3b ? PR3a : PR3b;
  // ---- aliased 2D layout (multiplicative): X, PM/PA and the x1 stage's output W start at word 0
  // (the x0 and x1 stages compute every line, the workgroup synchronises, then they write over
  // their inputs); W2 follows W
  static constexpr bool AL2 = ALIASv && D == 2;
  static constexpr int AL2a = X2 > P2 ? X2 : P2;
  static constexpr int AL2T = AL2a > m * T0 + m * TA ? AL2a : m * T0 + m * TA;
  static constexpr int total = D == 3 ? (PR ? PR3 : AL ? AL3 : A3 + B3) : (AL2 ? AL2T : A2 + B2);
  static constexpr int offX2 = AL2 ? 0 : A2, offP2 = 0, offW = AL2 ? 0 : A2, offW2 = AL2 ? m * T0 : 0;
  // 3D buffers
  static constexpr int offX = AL ? 0 : A3;
  static constexpr int offP = 0;
  static constexpr int offUV = AL ? 0 : A3;
  static constexpr int offW46 = PR ? 0 : AL ? UV3 : 0;  // W4 and W6
  static constexpr int offW57 = PR ? W46 : AL ? 0 : A3;  // W5 and W7
};

// A per-lane LDS offset the optimiser may not take apart.  Without it, base + i * stride inside an
// unrolled loop is re-associated into a fresh (quarter-rate) 32-bit multiply per element; behind
// this barrier each element is the base register plus a constant in the instruction's offset field.
__device__ __forceinline__ int lds_base(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// The constant tables re-derived through an opaque (but wave-uniform) zero
// offset: keeps the compiler from hoisting every table load out of a stage's
// task loop, which would pin more values in SGPRs than exist and spill them.
template <typename T>
__device__ __forceinline__ const DevTables<T>& tab_fresh(int k) {
  int z;
  asm volatile("s_mov_b32 %0, 0" : "=s"(z));
  return *reinterpret_cast<const DevTables<T>*>(reinterpret_cast<const char*>(&tab<T>(k)) + z);
}

// Eigenvector applications with the mirror parity of the patch eigenvectors (the 1D patch pair
// is symmetric under i -> m-1-i, so S[m-1-i][a] = par[a] S[i][a]): an even vector only sees
// v_i + v_{m-1-i}, an odd one v_i - v_{m-1-i}, which halves the multiply-adds.
// t[a] = sum_i S[i][a] v[i]
template <typename T, int K>
__device__ __forceinline__ void apply_st(const T (&v)[2 * K - 1], T (&t)[2 * K - 1]) {
  using PT = gen::PatchTables<T, K>;
  constexpr int m = 2 * K - 1, h = K - 1;
  T e[K], o[K];
#pragma unroll
  for (int i = 0; i < h; ++i) {
    e[i] = v[i] + v[m - 1 - i];
    o[i] = v[i] - v[m - 1 - i];
  }
  e[h] = v[h];
#pragma unroll
  for (int a = 0; a < m; ++a) {
    T s = T(0);
    if (a < K) {
#pragma unroll
      for (int i = 0; i <= h; ++i) s = fma_tab(PT::S[i * m + a], e[i], s);
    } else {
#pragma unroll
      for (int i = 0; i < h; ++i) s = fma_tab(PT::S[i * m + a], o[i], s);
    }
    t[a] = s;
  }
}

// w[i] = sum_a S[i][a] t[a]: w_i = E_i + O_i and w_{m-1-i} = E_i - O_i with E (O) the even (odd) part
template <typename T, int K>
__device__ __forceinline__ void apply_s(const T (&t)[2 * K - 1], T (&w)[2 * K - 1]) {
  using PT = gen::PatchTables<T, K>;
  constexpr int m = 2 * K - 1, h = K - 1;
#pragma unroll
  for (int i = 0; i <= h; ++i) {
    T ev = T(0), od = T(0);
#pragma unroll
    for (int a = 0; a < m; ++a) {
      if (a < K) {
        ev = fma_tab(PT::S[i * m + a], t[a], ev);
      } else if (i < h) {
        od = fma_tab(PT::S[i * m + a], t[a], od);
      }
    }
    w[i] = i < h ? ev + od : ev;  // the middle row has no odd part
    if (i < h) w[m - 1 - i] = ev - od;
  }
}

// ------------------------------------------------------------------ eigenbasis form
//
// The multiplicative pass computes x^I + A_j^{-1} (b^I - Abar_j x).  The local solver is exact, so the
// interior values cancel and the result is A_j^{-1} (b^I - A^{IB} x^B) (eq:A_ib_2d/3d): only the
// closure's boundary nodes enter.  Transformed by S^T along every axis, the boundary term needs no
// 1D matrix of the closure at all.  Write, along one axis, Mt = S^T M = [mu W mu'] and
// At = S^T A = Lambda Mt + [be 0 be'] (m x n; W the interior columns, mu/al/be the end columns, whose
// right-hand ones differ from the left by the eigenvectors' parity only).  Every boundary node belongs
// to one face: x0 faces own their whole closure, x1 faces the x0-interior part, x2 faces the x0- and
// x1-interior part.  A face F normal to axis a adds
//   al_a (x) P + mu_a (x) Q,   P = Mt (x) Mt F,   Q = (At (x) Mt + Mt (x) At) F
// (W in place of Mt along the axes where the face is interior only), so a patch costs six 2D face
// transforms, six multiply-adds per node in the eigenbasis, and the S^T / S transforms of the solve: in
// 3D Q4 about 18 k lane operations against 35 k of the form that contracts the whole closure with the
// 1D patch matrices.
// Rounding: that form's error is the cancellation in b - A x; this form's is relative to the values it
// transforms.  A constant c has A c = 0 on a patch's interior rows, so the pass runs on x^B - c and adds
// c at the end, c the mean of two opposite closure corners: the rounding is then relative to the
// variation of x over the patch.  Measured in an FP32 model of one step from the exact solution (error
// and residual, the closure form's in brackets): 2D Q3 32^2 3.0e-8, 5.8e-5 (6.7e-7, 1.6e-4); 2D Q7 64^2
// 3.0e-8, 1.7e-3 (1.4e-6, 3.8e-3); 3D Q3 16^3 1.4e-7, 3.3e-6 (6.9e-7, 3.6e-6); without c the residuals
// were 1.0-2.2 times the closure form's.

// t = Mt v for a closure line v (n values): the interior part through W, the ends through mu.  The
// even and odd end sums come back in Ee, Eo for the Lambda Mt + be form of At.
template <typename T, int K>
__device__ __forceinline__ void apply_mt(const T (&v)[2 * K + 1], T (&t)[2 * K - 1], T& Ee, T& Eo) {
  using PT = gen::PatchTables<T, K>;
  constexpr int m = 2 * K - 1, h = K - 1;
  T e[K], o[K];
#pragma unroll
  for (int i = 0; i < h; ++i) {
    e[i] = v[1 + i] + v[m - i];
    o[i] = v[1 + i] - v[m - i];
  }
  e[h] = v[1 + h];
  Ee = v[0] + v[2 * K];
  Eo = v[0] - v[2 * K];
#pragma unroll
  for (int a = 0; a < m; ++a) {
    T s = PT::mu[a] * (a < K ? +Ee : +Eo);
#pragma unroll
    for (int i = 0; i < (a < K ? K : h); ++i) s = fma(PT::W[a * m + i], a < K ? +e[i] : +o[i], s);
    t[a] = s;
  }
}

// t = W v (m values)
template <typename T, int K>
__device__ __forceinline__ void apply_w(const T (&v)[2 * K - 1], T (&t)[2 * K - 1]) {
  using PT = gen::PatchTables<T, K>;
  constexpr int m = 2 * K - 1, h = K - 1;
  T e[K], o[K];
#pragma unroll
  for (int i = 0; i < h; ++i) {
    e[i] = v[i] + v[m - 1 - i];
    o[i] = v[i] - v[m - 1 - i];
  }
  e[h] = v[h];
#pragma unroll
  for (int a = 0; a < m; ++a) {
    T s = T(0);
#pragma unroll
    for (int i = 0; i < (a < K ? K : h); ++i) s = fma(PT::W[a * m + i], a < K ? +e[i] : +o[i], s);
    t[a] = s;
  }
}

// Launch shape of the eigenbasis form: patches per workgroup, threads, and whether the buffers of
// consecutive stages share one LDS region (two more barriers, up to half the LDS).
template <int PPWv, int NTv, bool ALv>
struct EigShape {
  static constexpr int PPW = PPWv, NT = NTv;
  static constexpr bool AL = ALv;
};

constexpr int even_up(int v) { return v + (v & 1); }
constexpr int odd_up(int v) { return v | 1; }
constexpr int max_of(int a, int b) { return a > b ? a : b; }

// LDS of the 3D eigenbasis form (T words; "pairs" are two words moved by one access).  Stage A fills
// region A, stage B region B, stages C and D the transpose buffers W6 and W7.  Each buffer has the
// loop index of its reading stage outermost.
template <int K, typename SH>
struct EigLds3 {
  static constexpr int PPW = SH::PPW, n = 2 * K + 1, m = 2 * K - 1, mm = m * m, NF = 2 * PPW;
  static constexpr int SI1 = pad32(PPW * mm, m);     // BT [i1][q][a2][i0]
  static constexpr int SF0 = odd_up(NF * m);         // x0 faces, pairs [j1][q][end][a2]
  static constexpr int SF1 = odd_up(4 * PPW * m);    // x1 / x2 faces, pairs [i0][face][end][q][a2 or a1]
  static constexpr int offF0 = even_up(m * SI1), offF1 = offF0 + 2 * n * SF0;
  static constexpr int RA = offF1 + 2 * m * SF1;
  static constexpr int SI0 = pad32(PPW * mm, 1);     // W5 [i0][q][a2][a1]
  static constexpr int oP0 = even_up(m * SI0);       // pairs [q][end][a2][a1]
  static constexpr int oP1 = oP0 + 2 * NF * mm;      // pairs [a0][face][parity][q][a2 or a1]
  static constexpr int RB = oP1 + 2 * m * SF1;
  static constexpr int SA1 = pad32(PPW * mm, 1);     // W6 [a1][q][a2][i0]
  static constexpr int SA2 = pad32(PPW * mm, m);     // W7 [a2][i1][q][i0]
  static constexpr int W6 = even_up(m * SA1), W7 = even_up(m * SA2);
  static constexpr int A = max_of(RA, W6), B = max_of(RB, W7);
  static constexpr int offB = SH::AL ? 0 : A;
  static constexpr int offW6 = 0, offW7 = SH::AL ? W6 : A;
  static constexpr int offC = SH::AL ? max_of(max_of(RA, RB), W6 + W7) : A + B;  // the patches' constants
  static constexpr int total = offC + PPW;
};

// 3D eigenbasis pass.  Stages (tasks, the axis transformed):
//   A  b lines (i1, q, i0)       x2: S^T b                                  -> BT
//      rim columns of the patch closures in the (x0, x1) plane
//                                x2: (Mt, At) (x - c)                       -> x0 / x1 faces
//      x2-face lines (end, q, i0) x1: W (x - c) and its lambda multiple     -> x2 faces
//   B  b lines (q, a2, i0)       x1: S^T                                    -> W5
//      x0-face lines (q, end, a2) x1: P, Q                                  -> PQ0
//      x1- and x2-face lines (face, parity, q, a2 or a1)  x0: P, Q          -> PQ1
//   C  lines (q, a2, a1)         x0: S^T b, minus the face terms, 1/(lam2 + lam1 + lam0), S -> W6
//   D  lines (q, a2, i0)         x1: S                                      -> W7
//   E  lines (i1, q, i0)         x2: S, plus c, straight to global
// The lists of stages A and B are cut into whole waves per kind of task, so no wave mixes two kinds.
// tid: the thread's index in its team of SH::NT threads (the whole workgroup, or one of several that take
// different blocks and meet at the barriers); active: whether the team has a block.
// POISON: a non-finite old interior value makes the patch's result non-finite, as the residual form
// does (x^I enters through one multiply-add by zero per node); without it x^I is never read.
template <int K, typename T, bool POISON, typename SH, typename Win = Window<T>>
__device__ __forceinline__ void colour_pass_eig3(T* __restrict__ smem, const T* __restrict__ b, T* __restrict__ x,
                                                 long long n1d, int p0, int p1, int p2, int cnt0, int cnt1,
                                                 int groups0, T sol_scale, unsigned blk, int tid, bool active) {
  constexpr int n = 2 * K + 1, m = 2 * K - 1, mm = m * m;
  constexpr int PPW = SH::PPW, NT = SH::NT, NW = NT / 64;
  static_assert(NT % 64 == 0, "whole waves");
  using PT = gen::PatchTables<T, K>;
  using L = EigLds3<K, SH>;
  using T2 = typename Pair<T>::type;
  constexpr int NF = 2 * PPW;  // x0 faces

  const ColourBlock cb = colour_block<3, K, PPW>(blk, p0, p1, p2, cnt0, cnt1, groups0);
  const int P = active ? cb.count : 0;  // an idle team only meets the barriers
  const long long s0 = cb.s0, s1 = cb.s1, s2 = cb.s2;
  const long long n1d2 = n1d * n1d;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int seg = 2 * K * P + 1;  // valid closure columns along x0
  const int ld1 = (int)n1d;
  // windows at the closure corner of the first patch
  const unsigned span = (unsigned)(2 * K * (n1d2 + n1d) + seg) * (unsigned)sizeof(T);  // below 4 GiB (launcher)
  const Win xw(x + (s2 * n1d2 + s1 * n1d + s0), span), bw(b + (s2 * n1d2 + s1 * n1d + s0), span);
  // byte offsets of the closure's planes and of its rows, as scalars: derived again inside divergent
  // branches they would become per-lane values and every access a loop over the lanes
  unsigned pl[n], rw[m];
#pragma unroll
  for (int j = 0; j < n; ++j) pl[j] = __builtin_amdgcn_readfirstlane((unsigned)(j * n1d2) * (unsigned)sizeof(T));
#pragma unroll
  for (int i = 0; i < m; ++i) rw[i] = __builtin_amdgcn_readfirstlane((unsigned)(i * n1d) * (unsigned)sizeof(T));
  const bool lo0 = s0 == 0, hi0 = s0 + seg - 1 == n1d - 1;
  const bool lo1 = s1 == 0, hi1 = s1 + n - 1 == n1d - 1;
  const bool lo2 = s2 == 0, hi2 = s2 + n - 1 == n1d - 1;

  // the constant of patch q: the mean of its two extreme closure corners (a Dirichlet corner is 0)
  auto patch_constant = [&](int q) -> T {
    const unsigned lo = (unsigned)(2 * K * q) * (unsigned)sizeof(T);
    const unsigned hi = pl[2 * K] + (unsigned)(2 * K * (ld1 + q + 1)) * (unsigned)sizeof(T);
    const T u = xw.load(0, Win::masked((q == 0 && lo0) || lo1 || lo2, lo));
    const T v = xw.load(0, Win::masked((q == P - 1 && hi0) || hi1 || hi2, hi));
    return T(0.5) * (u + v);
  };

  // ---- A: the b lines' loads first, then the face lines, then the b transforms
  constexpr int NB = PPW * mm;                    // b lines
  constexpr int NR = 2 * PPW * (n + m);           // rim columns
  constexpr int NX = 2 * PPW * m;                 // x2-face lines
  constexpr int WB = (NB + 63) / 64, WR = (NR + 63) / 64, WX = (NX + 63) / 64;
  constexpr int RNDA = (WB + WR + WX + NW - 1) / NW;
  constexpr int RNB = (WB + NW - 1) / NW;         // rounds of the waves that hold b lines
  {
    T v[RNB][m], xp[RNB][m];
    auto b_line = [&](int u, int& i1, int& q, int& i0) -> bool {
      const int t = u * 64 + lane;
      i1 = div_small<PPW * m>(t);
      const int r = t - i1 * (PPW * m);
      q = div_small<m>(r);
      i0 = r - q * m;
      return t < NB && q < P;
    };
#pragma unroll
    for (int rr = 0; rr < RNB; ++rr) {
      const int u = rr * NW + wave;
      int i1, q, i0;
      if (u < WB && b_line(u, i1, q, i0)) {
        const unsigned off = (unsigned)((1 + i1) * ld1 + 2 * K * q + 1 + i0) * (unsigned)sizeof(T);
#pragma unroll
        for (int i = 0; i < m; ++i) v[rr][i] = bw.load(pl[1 + i], off);
        if constexpr (POISON) {
#pragma unroll
          for (int i = 0; i < m; ++i) xp[rr][i] = xw.load(pl[1 + i], off);
        }
      }
    }
    // face lines of wave-task u
    auto face_line = [&](int u) {
      if (u < WB + WR) {
        const int t = (u - WB) * 64 + lane;
        // the columns j1 = 0 and n - 1 of every patch, then its side columns (c = 0 and n - 1)
        int j1, q, c;
        if (t < 2 * PPW * n) {
          const int r = t < PPW * n ? t : t - PPW * n;
          j1 = t < PPW * n ? 0 : n - 1;
          q = div_small<n>(r);
          c = r - q * n;
        } else {
          const int g = t - 2 * PPW * n, jj = div_small<NF>(g), r = g - jj * NF;
          j1 = 1 + jj;
          q = r >> 1;
          c = (r & 1) * (n - 1);
        }
        if (t < NR && q < P) {
          const int end = c == 0 ? 0 : 1, col = 2 * K * q + c;
          const bool f0 = c == 0 || c == n - 1;  // x0 face, else x1 face
          // Dirichlet nodes count as 0 (the boundary entries of x are not read as values)
          const bool z = (col == 0 && lo0) || (col == seg - 1 && hi0) || (j1 == 0 && lo1) || (j1 == n - 1 && hi1);
          const unsigned off = Win::masked(z, (unsigned)(__mul24(j1, ld1) + col) * (unsigned)sizeof(T));
          T w[n], r[m], Ee, Eo;
#pragma unroll
          for (int j = 0; j < n; ++j) w[j] = xw.load(pl[j], off);
          const T cq = patch_constant(q);
          if (lo2) w[0] = T(0);
          if (hi2) w[n - 1] = T(0);
#pragma unroll
          for (int j = 0; j < n; ++j) w[j] -= cq;
          if (j1 == 0 && c == 0) smem[L::offC + q] = cq;
          apply_mt<T, K>(w, r, Ee, Eo);
          T2* F = reinterpret_cast<T2*>(smem) +
                  lds_base(f0 ? L::offF0 / 2 + j1 * L::SF0 + (2 * q + end) * m
                              : L::offF1 / 2 + (c - 1) * L::SF1 + ((j1 == 0 ? 0 : PPW) + q) * m);
#pragma unroll
          for (int a = 0; a < m; ++a) F[a] = T2{r[a], fma(PT::be[a], a < K ? +Ee : +Eo, PT::lam[a] * r[a])};
        }
      } else {
        const int t = (u - WB - WR) * 64 + lane;
        const int e = div_small<PPW * m>(t), g = t - e * (PPW * m), q = div_small<m>(g), i0 = g - q * m;
        if (t < NX && q < P) {
          const unsigned off =
              Win::masked(e == 0 ? lo2 : hi2,
                          (e == 0 ? 0u : pl[2 * K]) + (unsigned)(ld1 + 2 * K * q + 1 + i0) * (unsigned)sizeof(T));
          T w[m], r[m];
#pragma unroll
          for (int i = 0; i < m; ++i) w[i] = xw.load(rw[i], off);
          const T cq = patch_constant(q);
#pragma unroll
          for (int i = 0; i < m; ++i) w[i] -= cq;
          apply_w<T, K>(w, r);
          T2* F = reinterpret_cast<T2*>(smem) + lds_base(L::offF1 / 2 + i0 * L::SF1 + ((2 + e) * PPW + q) * m);
#pragma unroll
          for (int a = 0; a < m; ++a) F[a] = T2{r[a], PT::lam[a] * r[a]};
        }
      }
    };
#pragma unroll
    for (int rr = WB / NW; rr < RNDA; ++rr) {
      const int u = rr * NW + wave;
      if (u >= WB && u < WB + WR + WX) face_line(u);
    }
#pragma unroll
    for (int rr = 0; rr < RNB; ++rr) {
      const int u = rr * NW + wave;
      int i1, q, i0;
      if (u < WB && b_line(u, i1, q, i0)) {
        T r[m];
        if constexpr (POISON) {
#pragma unroll
          for (int i = 0; i < m; ++i) v[rr][0] = fma(T(0), xp[rr][i], v[rr][0]);
        }
        apply_st<T, K>(v[rr], r);
        const int ob = lds_base(i1 * L::SI1 + q * mm + i0);
#pragma unroll
        for (int a = 0; a < m; ++a) smem[ob + a * m] = r[a];
      }
    }
  }
  __syncthreads();
  // ---- B
  {
    constexpr int NF0 = NF * m, NF1 = 4 * PPW * m;
    constexpr int W0 = (NF0 + 63) / 64, W1 = (NF1 + 63) / 64, RNDB = (WB + W0 + W1 + NW - 1) / NW;
    const T2* F0 = reinterpret_cast<const T2*>(smem + L::offF0);
    const T2* F1 = reinterpret_cast<const T2*>(smem + L::offF1);
    T* W5 = smem + L::offB;
    T2* PQ0 = reinterpret_cast<T2*>(smem + L::offB + L::oP0);
    T2* PQ1 = reinterpret_cast<T2*>(smem + L::offB + L::oP1);
    T rb[RNB][m], r0[RNDB][m], r1[RNDB][m];
    // patches past the last one: whatever the buffers hold, never stored to global
    auto b_work = [&](int u, T (&a0)[m]) {
      const int t = u * 64 + lane;
      if (u < WB && t < NB) {
        T in[m];
#pragma unroll
        for (int i = 0; i < m; ++i) in[i] = smem[i * L::SI1 + t];
        apply_st<T, K>(in, a0);
      }
    };
    auto b_put = [&](int u, const T (&a0)[m]) {
      const int t = u * 64 + lane;
      if (u < WB && t < NB) {
        const int r = div_small<m>(t), i0 = t - r * m;  // r = q * m + a2
        const int ob = lds_base(i0 * L::SI0 + r * m);
#pragma unroll
        for (int a = 0; a < m; ++a) W5[ob + a] = a0[a];
      }
    };
    // face task u of the wave: P in a0, Q in a1
    auto work = [&](int u, T (&a0)[m], T (&a1)[m]) {
      if (u < WB) return;
      if (u < WB + W0) {
        const int t = (u - WB) * 64 + lane;
        if (t < NF0) {
          T mv[n], av[n], Ee, Eo, Fe, Fo, q[m];
#pragma unroll
          for (int j = 0; j < n; ++j) {
            const T2 w = F0[j * L::SF0 + t];
            mv[j] = w.x;
            av[j] = w.y;
          }
          apply_mt<T, K>(mv, a0, Ee, Eo);
          apply_mt<T, K>(av, q, Fe, Fo);
#pragma unroll
          for (int a = 0; a < m; ++a) a1[a] = fma(PT::be[a], a < K ? +Ee : +Eo, fma(PT::lam[a], a0[a], q[a]));
        }
      } else if (u < WB + W0 + W1) {
        const int t = (u - WB - W0) * 64 + lane;
        if (t < NF1) {
          // (face, parity, q, a): the sum or difference of the face's two ends
          const int g = div_small<PPW * m>(t), par = g & 1, base = (g - par) * (PPW * m) + (t - g * (PPW * m));
          const T sg = par ? T(-1) : T(1);
          T mv[m], av[m], q[m];
#pragma unroll
          for (int i = 0; i < m; ++i) {
            const T2 lf = F1[i * L::SF1 + base], rt = F1[i * L::SF1 + base + PPW * m];
            mv[i] = fma(sg, rt.x, lf.x);
            av[i] = fma(sg, rt.y, lf.y);
          }
          apply_w<T, K>(mv, a0);
          apply_w<T, K>(av, q);
#pragma unroll
          for (int a = 0; a < m; ++a) a1[a] = fma(PT::lam[a], a0[a], q[a]);
        }
      }
    };
    auto put = [&](int u, const T (&a0)[m], const T (&a1)[m]) {
      if (u < WB) return;
      if (u < WB + W0) {
        const int t = (u - WB) * 64 + lane;
        if (t < NF0) {
          T2* d = PQ0 + lds_base(t * m);
#pragma unroll
          for (int a = 0; a < m; ++a) d[a] = T2{a0[a], a1[a]};
        }
      } else if (u < WB + W0 + W1) {
        const int t = (u - WB - W0) * 64 + lane;
        if (t < NF1) {
          T2* d = PQ1 + lds_base(t);
#pragma unroll
          for (int a = 0; a < m; ++a) d[a * L::SF1] = T2{a0[a], a1[a]};
        }
      }
    };
    if constexpr (SH::AL) {
#pragma unroll
      for (int rr = 0; rr < RNB; ++rr) b_work(rr * NW + wave, rb[rr]);
#pragma unroll
      for (int rr = WB / NW; rr < RNDB; ++rr) work(rr * NW + wave, r0[rr], r1[rr]);
      __syncthreads();
#pragma unroll
      for (int rr = 0; rr < RNB; ++rr) b_put(rr * NW + wave, rb[rr]);
#pragma unroll
      for (int rr = WB / NW; rr < RNDB; ++rr) put(rr * NW + wave, r0[rr], r1[rr]);
    } else {
#pragma unroll
      for (int rr = 0; rr < RNB; ++rr) {
        b_work(rr * NW + wave, rb[0]);
        b_put(rr * NW + wave, rb[0]);
      }
#pragma unroll
      for (int rr = WB / NW; rr < RNDB; ++rr) {
        work(rr * NW + wave, r0[0], r1[0]);
        put(rr * NW + wave, r0[0], r1[0]);
      }
    }
  }
  // ---- C
  constexpr int RC = (NB + NT - 1) / NT;
  {
    const DevTables<T>& tb = tab_fresh<T>(K);
    const T* W5 = smem + L::offB;
    const T2* PQ0 = reinterpret_cast<const T2*>(smem + L::offB + L::oP0);
    const T2* PQ1 = reinterpret_cast<const T2*>(smem + L::offB + L::oP1);
    T* W6 = smem + L::offW6;
    T w[RC][m], iv[RC][m], c1[RC][2], c2[RC][2];
    // the lane's table entries, fetched before the barrier
#pragma unroll
    for (int rr = 0; rr < RC; ++rr) {
      const int t = rr * NT + tid, r = t - div_small<mm>(t) * mm, a2 = div_small<m>(r), a1 = r - a2 * m;
#pragma unroll
      for (int a = 0; a < m; ++a) iv[rr][a] = tb.inv3[r * m + a];
      c1[rr][0] = tb.al[a1];
      c1[rr][1] = tb.mu[a1];
      c2[rr][0] = tb.al[a2];
      c2[rr][1] = tb.mu[a2];
    }
    __syncthreads();
    auto put = [&](int t, const T (&v)[m]) {
      const int q = div_small<mm>(t), r = t - q * mm, a2 = div_small<m>(r), a1 = r - a2 * m;
      const int ob = lds_base(a1 * L::SA1 + q * mm + a2 * m);
#pragma unroll
      for (int i = 0; i < m; ++i) W6[ob + i] = v[i];
    };
#pragma unroll
    for (int rr = 0; rr < RC; ++rr) {
      const int t = rr * NT + tid;
      const int q = div_small<mm>(t), r = t - q * mm, a2 = div_small<m>(r), a1 = r - a2 * m;
      if (t < NB && q < P) {
        T in[m], z[m];
#pragma unroll
        for (int i = 0; i < m; ++i) in[i] = W5[i * L::SI0 + t];
        apply_st<T, K>(in, z);
        const T2 f0 = PQ0[t + q * mm], f1 = PQ0[t + (q + 1) * mm];
        const T pe = f0.x + f1.x, po = f0.x - f1.x, qe = f0.y + f1.y, qo = f0.y - f1.y;
        const T2* F1 = PQ1 + lds_base((a1 < K ? 0 : PPW * m) + q * m + a2);
        const T2* F2 = PQ1 + lds_base((a2 < K ? 2 : 3) * PPW * m + q * m + a1);
#pragma unroll
        for (int a = 0; a < m; ++a) {
          const T2 u1 = F1[a * L::SF1], u2 = F2[a * L::SF1];
          T g = PT::al[a] * (a < K ? +pe : +po);
          g = fma(PT::mu[a], a < K ? +qe : +qo, g);
          g = fma(c1[rr][0], u1.x, g);
          g = fma(c1[rr][1], u1.y, g);
          g = fma(c2[rr][0], u2.x, g);
          g = fma(c2[rr][1], u2.y, g);
          z[a] = fma(sol_scale, z[a], -g) * iv[rr][a];
        }
        apply_s<T, K>(z, w[rr]);
        if constexpr (!SH::AL) put(t, w[rr]);
      }
    }
    if constexpr (SH::AL) {
      __syncthreads();
#pragma unroll
      for (int rr = 0; rr < RC; ++rr) {
        const int t = rr * NT + tid;
        if (t < NB && div_small<mm>(t) < P) put(t, w[rr]);
      }
    }
  }
  __syncthreads();
  // ---- D
  {
    const T* W6 = smem + L::offW6;
    T* W7 = smem + L::offW7;
#pragma unroll
    for (int rr = 0; rr < RC; ++rr) {
      const int t = rr * NT + tid;
      const int q = div_small<mm>(t), r = t - q * mm, a2 = div_small<m>(r), i0 = r - a2 * m;
      if (t < NB && q < P) {
        T in[m], w[m];
#pragma unroll
        for (int a = 0; a < m; ++a) in[a] = W6[a * L::SA1 + t];
        apply_s<T, K>(in, w);
        const int ob = lds_base(a2 * L::SA2 + q * m + i0);
#pragma unroll
        for (int i = 0; i < m; ++i) W7[ob + i * (PPW * m)] = w[i];
      }
    }
  }
  __syncthreads();
  // ---- E
  {
    const T* W7 = smem + L::offW7;
#pragma unroll
    for (int rr = 0; rr < RC; ++rr) {
      const int t = rr * NT + tid;
      const int i1 = div_small<PPW * m>(t), r = t - i1 * (PPW * m), q = div_small<m>(r), i0 = r - q * m;
      if (t < NB && q < P) {
        T in[m], w[m];
#pragma unroll
        for (int a = 0; a < m; ++a) in[a] = W7[a * L::SA2 + t];
        const T cq = smem[L::offC + q];
        apply_s<T, K>(in, w);
        const unsigned off = (unsigned)((1 + i1) * ld1 + 2 * K * q + 1 + i0) * (unsigned)sizeof(T);
#pragma unroll
        for (int i = 0; i < m; ++i) xw.store(pl[1 + i], off, w[i] + cq);
      }
    }
  }
}

// LDS of the 2D eigenbasis form.
template <int K, typename SH>
struct EigLds2 {
  static constexpr int PPW = SH::PPW, n = 2 * K + 1, m = 2 * K - 1, NF = 2 * PPW;
  static constexpr int T0 = pad32(PPW * m, 1);        // W [i0][q][a1]
  static constexpr int oP0 = even_up(m * T0);         // x0 faces, pairs (P, Q) [q][end][a1]
  static constexpr int SP1 = odd_up(PPW);
  static constexpr int oP1 = oP0 + 2 * NF * m;        // x1 faces, pairs (low end, high end) [a0][q]
  static constexpr int RA = oP1 + 2 * m * SP1;
  static constexpr int TA = pad32(PPW * m, 1);        // W2 [a1][q][i0]
  static constexpr int offW2 = SH::AL ? 0 : RA;
  static constexpr int offC = SH::AL ? max_of(RA, m * TA) : RA + m * TA;  // the patches' constants
  static constexpr int total = offC + PPW;
};

// 2D eigenbasis pass.
//   A  b lines (q, i0)            x1: S^T b                                 -> W
//      face lines of x - c: x0 faces (q, end) along x1 (P = Mt F, Q = At F), x1 faces (end, q) along x0
//      (W F)                                                              -> PQ0, P1
//   B  lines (q, a1)              x0: S^T b, minus the face terms, 1/(lam1 + lam0), S -> W2
//   C  lines (q, i0)              x1: S, plus c, straight to global
template <int K, typename T, bool POISON, typename SH, typename Win = Window<T>>
__device__ __forceinline__ void colour_pass_eig2(T* __restrict__ smem, const T* __restrict__ b, T* __restrict__ x,
                                                 long long n1d, int p0, int p1, int cnt0, int cnt1, int groups0,
                                                 T sol_scale, unsigned blk, int tid, bool active) {
  constexpr int n = 2 * K + 1, m = 2 * K - 1;
  constexpr int PPW = SH::PPW, NT = SH::NT, NW = NT / 64;
  static_assert(NT % 64 == 0, "whole waves");
  using PT = gen::PatchTables<T, K>;
  using L = EigLds2<K, SH>;
  using T2 = typename Pair<T>::type;
  constexpr int NF = 2 * PPW;  // x0 faces

  const ColourBlock cb = colour_block<2, K, PPW>(blk, p0, p1, 0, cnt0, cnt1, groups0);
  const int P = active ? cb.count : 0;  // an idle team only meets the barriers
  const long long s0 = cb.s0, s1 = cb.s1;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int seg = 2 * K * P + 1;
  const int ld1 = (int)n1d;
  // windows at the closure corner of the first patch
  const unsigned span = (unsigned)(2 * K * n1d + seg) * (unsigned)sizeof(T);  // below 4 GiB (launcher)
  const Win xw(x + (s1 * n1d + s0), span), bw(b + (s1 * n1d + s0), span);
  unsigned rw[m];  // byte offsets of the interior rows (scalars, as in the 3D form)
#pragma unroll
  for (int i = 0; i < m; ++i) rw[i] = __builtin_amdgcn_readfirstlane((unsigned)((1 + i) * n1d) * (unsigned)sizeof(T));
  const bool lo0 = s0 == 0, hi0 = s0 + seg - 1 == n1d - 1;
  const bool lo1 = s1 == 0, hi1 = s1 + n - 1 == n1d - 1;

  constexpr int NB = PPW * m, NX = NF + 2 * PPW;  // b lines, face lines
  constexpr int WB = (NB + 63) / 64, WX = (NX + 63) / 64, RNDA = (WB + WX + NW - 1) / NW;
  T* W = smem;
  T2* PQ0 = reinterpret_cast<T2*>(smem + L::oP0);
  {
    T v[RNDA][n], xp[RNDA][m], cq[RNDA];
    // face line of wave-task u: x0 face (q, end e) or x1 face (end e, q)
    auto face_line = [&](int u, bool& f0, int& q, int& e) -> bool {
      const int t = (u - WB) * 64 + lane, g = t - NF;
      f0 = t < NF;
      e = f0 ? t & 1 : g >= PPW ? 1 : 0;
      q = f0 ? t >> 1 : g - e * PPW;
      return t < NX && q < P;
    };
#pragma unroll
    for (int rr = 0; rr < RNDA; ++rr) {
      const int u = rr * NW + wave;
      if (u < WB) {
        const int t = u * 64 + lane, q = div_small<m>(t), i0 = t - q * m;
        if (t < NB && q < P) {
          const unsigned off = (unsigned)(2 * K * q + 1 + i0) * (unsigned)sizeof(T);
#pragma unroll
          for (int i = 0; i < m; ++i) v[rr][i] = bw.load(rw[i], off);
          if constexpr (POISON) {
#pragma unroll
            for (int i = 0; i < m; ++i) xp[rr][i] = xw.load(rw[i], off);
          }
        }
      } else if (u < WB + WX) {
        bool f0;
        int q, e;
        if (face_line(u, f0, q, e)) {
          // node j of the line at off + j * stride
          const unsigned off = (unsigned)(2 * K * (f0 ? q + e : q + e * ld1)) * (unsigned)sizeof(T);
          const unsigned st = (unsigned)(f0 ? ld1 : 1) * (unsigned)sizeof(T);
#pragma unroll
          for (int j = 0; j < n; ++j) v[rr][j] = xw.load(0, off + (unsigned)j * st);
          // the mean of the patch's two extreme closure corners (a Dirichlet corner is 0)
          const unsigned hi = (unsigned)(2 * K * (ld1 + q + 1)) * (unsigned)sizeof(T);
          cq[rr] = T(0.5) * (xw.load(0, Win::masked((q == 0 && lo0) || lo1, (unsigned)(2 * K * q) * (unsigned)sizeof(T))) +
                             xw.load(0, Win::masked((q == P - 1 && hi0) || hi1, hi)));
        }
      }
    }
#pragma unroll
    for (int rr = 0; rr < RNDA; ++rr) {
      const int u = rr * NW + wave;
      if (u < WB) {
        const int t = u * 64 + lane, q = div_small<m>(t), i0 = t - q * m;
        if (t < NB && q < P) {
          T w[m], s[m];
#pragma unroll
          for (int i = 0; i < m; ++i) {
            w[i] = v[rr][i];
            if constexpr (POISON) w[0] = fma(T(0), xp[rr][i], w[0]);
          }
          apply_st<T, K>(w, s);
          const int ob = lds_base(i0 * L::T0 + q * m);
#pragma unroll
          for (int a = 0; a < m; ++a) W[ob + a] = s[a];
        }
      } else if (u < WB + WX) {
        bool f0;
        int q, e;
        if (face_line(u, f0, q, e)) {
          const bool z = f0 ? (q + e == 0 && lo0) || (q + e == P && hi0) : e ? hi1 : lo1;
          T w[n], s[m], Ee, Eo;
#pragma unroll
          for (int j = 0; j < n; ++j) w[j] = z ? T(0) : v[rr][j];
          if (lo1) w[0] = f0 ? T(0) : w[0];
          if (hi1) w[n - 1] = f0 ? T(0) : w[n - 1];
#pragma unroll
          for (int j = 0; j < n; ++j) w[j] -= cq[rr];
          if (!f0) w[0] = w[n - 1] = T(0);  // the corners belong to the x0 faces
          if (f0 && e == 0) smem[L::offC + q] = cq[rr];
          apply_mt<T, K>(w, s, Ee, Eo);
          if (f0) {
            T2* d = PQ0 + lds_base((2 * q + e) * m);
#pragma unroll
            for (int a = 0; a < m; ++a) d[a] = T2{s[a], fma(PT::be[a], a < K ? +Ee : +Eo, PT::lam[a] * s[a])};
          } else {
            T* d = smem + lds_base(L::oP1 + 2 * q + e);
#pragma unroll
            for (int a = 0; a < m; ++a) d[a * 2 * L::SP1] = s[a];
          }
        }
      }
    }
  }
  // ---- B
  constexpr int RC = (NB + NT - 1) / NT;
  {
    const DevTables<T>& tb = tab_fresh<T>(K);
    T* W2 = smem + L::offW2;
    T w[RC][m], iv[RC][m], c1[RC][2];
#pragma unroll
    for (int rr = 0; rr < RC; ++rr) {
      const int t = rr * NT + tid, a1 = t - div_small<m>(t) * m;
#pragma unroll
      for (int a = 0; a < m; ++a) iv[rr][a] = tb.inv2[a1 * m + a];
      c1[rr][0] = tb.al[a1];
      c1[rr][1] = tb.mu[a1];
    }
    __syncthreads();
    auto put = [&](int t, const T (&v)[m]) {
      const int q = div_small<m>(t), a1 = t - q * m;
      const int ob = lds_base(a1 * L::TA + q * m);
#pragma unroll
      for (int i = 0; i < m; ++i) W2[ob + i] = v[i];
    };
#pragma unroll
    for (int rr = 0; rr < RC; ++rr) {
      const int t = rr * NT + tid, q = div_small<m>(t), a1 = t - q * m;
      if (t < NB && q < P) {
        T in[m], z[m];
#pragma unroll
        for (int i = 0; i < m; ++i) in[i] = W[i * L::T0 + t];
        apply_st<T, K>(in, z);
        const T2 f0 = PQ0[t + q * m], f1 = PQ0[t + (q + 1) * m];
        const T pe = f0.x + f1.x, po = f0.x - f1.x, qe = f0.y + f1.y, qo = f0.y - f1.y;
        const T sg = a1 < K ? T(1) : T(-1);
        const T2* F1 = reinterpret_cast<const T2*>(smem + L::oP1) + lds_base(q);
#pragma unroll
        for (int a = 0; a < m; ++a) {
          const T2 e = F1[a * L::SP1];
          T g = PT::al[a] * (a < K ? +pe : +po);
          g = fma(PT::mu[a], a < K ? +qe : +qo, g);
          g = fma(fma(c1[rr][1], PT::lam[a], c1[rr][0]), fma(sg, e.y, e.x), g);
          z[a] = fma(sol_scale, z[a], -g) * iv[rr][a];
        }
        apply_s<T, K>(z, w[rr]);
        if constexpr (!SH::AL) put(t, w[rr]);
      }
    }
    if constexpr (SH::AL) {
      __syncthreads();
#pragma unroll
      for (int rr = 0; rr < RC; ++rr) {
        const int t = rr * NT + tid;
        if (t < NB && div_small<m>(t) < P) put(t, w[rr]);
      }
    }
  }
  __syncthreads();
  // ---- C
  {
    const T* W2 = smem + L::offW2;
#pragma unroll
    for (int rr = 0; rr < RC; ++rr) {
      const int t = rr * NT + tid, q = div_small<m>(t), i0 = t - q * m;
      if (t < NB && q < P) {
        T in[m], w[m];
#pragma unroll
        for (int a = 0; a < m; ++a) in[a] = W2[a * L::TA + t];
        const T cq = smem[L::offC + q];
        apply_s<T, K>(in, w);
        const unsigned off = (unsigned)(2 * K * q + 1 + i0) * (unsigned)sizeof(T);
#pragma unroll
        for (int i = 0; i < m; ++i) xw.store(rw[i], off, w[i] + cq);
      }
    }
  }
}

// Degree 1: a patch has one interior node, so the pass is a stencil (9 or 27 points) with one thread per
// patch, PPW consecutive patches along x0 per one-wave workgroup, and neither LDS nor a barrier.  The
// residual b - h^(d-2) Abar x is summed row by row from the 1D patch rows (Sec. 3.1.1), then
// x^I += residual / (h^(d-2) diagonal); without OLD (Boundary mode) the old x^I counts as 0.
template <int D, typename T, bool OLD, int PPW, typename Win = Window<T>>
__device__ __forceinline__ void colour_pass_q1(const T* __restrict__ b, T* __restrict__ x, long long n1d, int p0, int p1,
                                               int p2, int cnt0, int cnt1, int groups0, T res_scale, T sol_scale,
                                               unsigned blk, int tid, bool active) {
  using PT = gen::PatchTables<T, 1>;
  constexpr int n = 3, J2 = D == 3 ? n : 1;
  const ColourBlock cb = colour_block<D, 1, PPW>(blk, p0, p1, p2, cnt0, cnt1, groups0);
  const int q = tid, seg = 2 * cb.count + 1;
  const long long n1d2 = n1d * n1d, origin = (D == 3 ? cb.s2 * n1d2 : 0) + cb.s1 * n1d + cb.s0;
  const unsigned span = (unsigned)((D == 3 ? 2 * n1d2 : 0) + 2 * n1d + seg) * (unsigned)sizeof(T);
  const Win xw(x + origin, span), bw(b + origin, span);
  const bool lo0 = cb.s0 == 0, hi0 = cb.s0 + seg - 1 == n1d - 1;
  const bool edge1[2] = {cb.s1 == 0, cb.s1 + 2 == n1d - 1};
  const bool edge2[2] = {D == 3 && cb.s2 == 0, D == 3 && cb.s2 + 2 == n1d - 1};
  if (!active || q >= cb.count) return;
  // the patch's columns 2q, 2q + 1, 2q + 2; Dirichlet columns read as 0
  unsigned off[n];
#pragma unroll
  for (int c = 0; c < n; ++c) off[c] = (unsigned)(2 * q + c) * (unsigned)sizeof(T);
  if (q == 0 && lo0) off[0] = Win::masked(true, off[0]);
  if (q == cb.count - 1 && hi0) off[2] = Win::masked(true, off[2]);
  const unsigned centre = (unsigned)((D == 3 ? n1d2 : 0) + n1d) * (unsigned)sizeof(T);
  const T bv = bw.load(centre, off[1]);
  T v[J2][n][n];
#pragma unroll
  for (int j2 = 0; j2 < J2; ++j2)
#pragma unroll
    for (int j1 = 0; j1 < n; ++j1) {
      const unsigned row = (unsigned)((D == 3 ? j2 * n1d2 : 0) + j1 * n1d) * (unsigned)sizeof(T);
      const bool dirichlet = (j1 == 0 && edge1[0]) || (j1 == 2 && edge1[1]) ||
                             (D == 3 && ((j2 == 0 && edge2[0]) || (j2 == 2 && edge2[1])));
#pragma unroll
      for (int c = 0; c < n; ++c) v[j2][j1][c] = dirichlet ? T(0) : xw.load(row, off[c]);
    }
  constexpr int jc = D == 3 ? 1 : 0;
  const T old = v[jc][1][1];
  if (!OLD) v[jc][1][1] = T(0);
  T sum = T(0);
#pragma unroll
  for (int j2 = 0; j2 < J2; ++j2) {
    T u = T(0), w = T(0);
#pragma unroll
    for (int j1 = 0; j1 < n; ++j1) {
      T pm = T(0), pa = T(0);
#pragma unroll
      for (int c = 0; c < n; ++c) {
        pm = fma(PT::Mc[c], v[j2][j1][c], pm);
        pa = fma(PT::Ac[c], v[j2][j1][c], pa);
      }
      u = fma(PT::Mc[j1], pm, u);
      w = fma(PT::Ac[j1], pm, fma(PT::Mc[j1], pa, w));
    }
    sum = D == 3 ? fma(PT::Ac[j2], u, fma(PT::Mc[j2], w, sum)) : w;
  }
  constexpr T inv = (T)(1.0 / (D * 2.0 * (D == 3 ? 4.0 / 9.0 : 2.0 / 3.0)));  // patch matrix of h = 1: d A M^(d-1)
  const T r = fma(-res_scale, sum, bv) * inv;
  xw.store(centre, off[1], OLD ? fma(sol_scale, r, old) : sol_scale * r);
}

// Launch shapes of the multiplicative and Boundary passes per (dim, degree, precision): Large, and the
// Small one that a launch takes when Large would give fewer than kEigWaves waves.  Both columns are
// the fastest of 5-20 (patches, threads, layout) per row over the levels they serve; patches per
// workgroup that divide the power-of-two rows leave no slot idle.
// Measured, back-to-back passes of a step, us, the residual form's in brackets, FP32 / FP64: 3D degree 3, 64^3
// cells 20.2 (23.2) / 29.9 (32.3); degree 4, 64^3 38.5 (46.5) / 73.4 (83.7); degree 5, 32^3 13.3 (16.9) / 24.1
// (27.7); degree 6, 32^3 21.7 (25.9) / 38.8 (47.7); degree 7, 32^3 33.7 (40.9) / 62.3 (78.1); 2D 512^2 degree 5
// 16.3 (17.9) / 27.3 (31.5), degree 6 22.2 (24.4) / 38.7 (47.9), degree 7 27.9 (31.4) / 52.1 (65.5).
// 3D degree 4 FP32 issues 14.9-16.3 M vector instructions a pass (18.8 M), 77% of its cycles, and its LDS pipe is
// busy 80% of them; the FP64 passes run at 4.6-5.1 TB/s of closure-once traffic.
template <int PPWv>
struct Q1Shape {
  static constexpr int PPW = PPWv, NT = PPWv;
};
template <int D, int K, typename T>
struct EigShapes;
template <typename T> struct EigShapes<3, 1, T> { using Large = Q1Shape<64>; using Small = Large; };
template <typename T> struct EigShapes<3, 2, T> { using Large = EigShape<16, 256, true>; using Small = EigShape<4, 192, false>; };
template <typename T> struct EigShapes<3, 3, T> { using Large = EigShape<5, 192, true>; using Small = EigShape<2, 192, false>; };
template <> struct EigShapes<3, 4, float> { using Large = EigShape<4, 256, true>; using Small = EigShape<1, 192, false>; };
template <> struct EigShapes<3, 4, double> { using Large = EigShape<2, 128, true>; using Small = EigShape<1, 192, false>; };
template <typename T> struct EigShapes<3, 5, T> { using Large = EigShape<3, 256, true>; using Small = EigShape<1, 256, false>; };
template <typename T> struct EigShapes<3, 6, T> { using Large = EigShape<2, 256, true>; using Small = EigShape<1, 256, false>; };
template <> struct EigShapes<3, 7, float> { using Large = EigShape<1, 320, true>; using Small = EigShape<1, 320, false>; };
template <> struct EigShapes<3, 7, double> { using Large = EigShape<1, 192, true>; using Small = EigShape<1, 320, false>; };
template <typename T> struct EigShapes<2, 1, T> { using Large = Q1Shape<64>; using Small = Large; };
template <typename T> struct EigShapes<2, 2, T> { using Large = EigShape<42, 192, false>; using Small = EigShape<8, 128, false>; };
template <typename T> struct EigShapes<2, 3, T> { using Large = EigShape<32, 256, false>; using Small = EigShape<8, 128, false>; };
template <typename T> struct EigShapes<2, 4, T> { using Large = EigShape<8, 128, false>; using Small = EigShape<4, 128, false>; };
template <typename T> struct EigShapes<2, 5, T> { using Large = EigShape<14, 192, false>; using Small = EigShape<4, 128, false>; };
template <typename T> struct EigShapes<2, 6, T> { using Large = EigShape<11, 192, false>; using Small = EigShape<4, 128, false>; };
template <typename T> struct EigShapes<2, 7, T> { using Large = EigShape<9, 192, true>; using Small = EigShape<4, 128, false>; };
constexpr long long kEigWaves = 1100;
// 3D degree 7 in FP32 takes three patches per workgroup where the iterate and the right-hand side do not fit the
// 256 MB last-level cache together: longer row segments for HBM (64^3 cells: 254 us a pass against 274; on 32^3,
// which fits, 36.1 against 30.7).
constexpr long long kLastLevelCache = 256LL << 20;
template <int D, int K, typename T>
struct FarShape {
  using type = void;
};
template <> struct FarShape<3, 7, float> { using type = EigShape<3, 512, true>; };
// ------------------------------------------------------------------ passes without a residual
//
// Additive pass x^I += A_j^{-1} b^I; ZERO: the first colour of a step on x = 0 (kModeZero), which stores
// A_j^{-1} b^I on the patch interiors and 0 on the rest of its closures and reads no x.  The eigenbasis pass
// without faces: the same line stages, row-ordered global accesses and team arguments.
template <int D, int K, typename SH>
struct AddLds {
  static constexpr int PPW = SH::PPW, m = 2 * K - 1, mm = m * m;
  static constexpr int SI1 = pad32(PPW * mm, m);  // BT [i1][q][a2][i0]
  static constexpr int SI0 = pad32(PPW * mm, 1);  // W5 [i0][q][a2][a1]
  static constexpr int SA1 = pad32(PPW * mm, 1);  // W6 [a1][q][a2][i0]
  static constexpr int SA2 = pad32(PPW * mm, m);  // W7 [a2][i1][q][i0]
  static constexpr int T0 = pad32(PPW * m, 1);    // 2D: W [i0][q][a1], W2 [a1][q][i0]
  static constexpr int A = D == 3 ? m * max_of(SI1, SA1) : m * T0, B = D == 3 ? m * max_of(SI0, SA2) : m * T0;
  static constexpr int total = A + B;
};

template <int D, int K, typename T, bool ZERO, typename SH>
__device__ __forceinline__ void colour_pass_add(T* __restrict__ smem, const T* __restrict__ b, T* __restrict__ x,
                                                long long n1d, int p0, int p1, int p2, int cnt0, int cnt1, int groups0,
                                                T sol_scale, unsigned blk, int tid, bool active) {
  constexpr int n = 2 * K + 1, m = 2 * K - 1, mm = m * m;
  constexpr int PPW = SH::PPW, NT = SH::NT, NB = D == 3 ? PPW * mm : PPW * m, RC = (NB + NT - 1) / NT;
  using L = AddLds<D, K, SH>;
  const ColourBlock cb = colour_block<D, K, PPW>(blk, p0, p1, p2, cnt0, cnt1, groups0);
  const int P = active ? cb.count : 0;
  const long long n1d2 = n1d * n1d, origin = (D == 3 ? cb.s2 * n1d2 : 0) + cb.s1 * n1d + cb.s0;
  const int seg = 2 * K * P + 1, ld1 = (int)n1d;
  const unsigned span = (unsigned)((D == 3 ? 2 * K * n1d2 : 0) + 2 * K * n1d + seg) * (unsigned)sizeof(T);
  const Window<T> xw(x + origin, span), bw(b + origin, span);
  // interior planes (3D) or rows (2D) along the slowest axis
  unsigned pl[m];
#pragma unroll
  for (int i = 0; i < m; ++i)
    pl[i] = __builtin_amdgcn_readfirstlane((unsigned)((1 + i) * (D == 3 ? n1d2 : n1d)) * (unsigned)sizeof(T));
  // line t of the slowest axis, (i1, q, i0) in 3D and (q, i0) in 2D: byte offset inside its plane or row
  auto line = [&](int t, int& q, int& i1, int& i0, unsigned& off) -> bool {
    if constexpr (D == 3) {
      i1 = div_small<PPW * m>(t);
      const int r = t - i1 * (PPW * m);
      q = div_small<m>(r);
      i0 = r - q * m;
      off = (unsigned)((1 + i1) * ld1 + 2 * K * q + 1 + i0) * (unsigned)sizeof(T);
    } else {
      q = div_small<m>(t);
      i1 = 0;
      i0 = t - q * m;
      off = (unsigned)(2 * K * q + 1 + i0) * (unsigned)sizeof(T);
    }
    return t < NB && q < P;
  };
  T v[RC][m], xo[RC][m], iv[RC][m];
#pragma unroll
  for (int rr = 0; rr < RC; ++rr) {
    int q, i1, i0;
    unsigned off;
    if (line(rr * NT + tid, q, i1, i0, off)) {
#pragma unroll
      for (int i = 0; i < m; ++i) v[rr][i] = bw.load(pl[i], off);
      if constexpr (!ZERO) {
#pragma unroll
        for (int i = 0; i < m; ++i) xo[rr][i] = xw.load(pl[i], off);
      }
    }
  }
  if constexpr (ZERO) {
    // 0 on every closure node that is not a patch interior (neighbouring workgroups write the same zeros on shared
    // faces; no interior of the colour lies there): the face rows whole, on the others the columns between patches
    constexpr int RS = 2 * K * PPW + 1, NFR = D == 3 ? 4 * (n - 1) : 2, NIR = D == 3 ? mm : m;
    constexpr int NZF = NFR * RS, NZ = NZF + NIR * (PPW + 1);
    for (int w = tid; w < NZ && P > 0; w += NT) {
      int j1, j2 = 0, c;
      if (w < NZF) {
        const int f = w / RS;
        c = w - f * RS;
        if constexpr (D == 3) {
          if (f < 2 * n) {
            j2 = f < n ? 0 : n - 1;
            j1 = f < n ? f : f - n;
          } else {
            j2 = 1 + (f - 2 * n) / 2;
            j1 = (f & 1) ? n - 1 : 0;  // f - 2n and f have the same parity (2n even)
          }
        } else {
          j1 = f == 0 ? 0 : n - 1;
        }
      } else {
        const int u = w - NZF, r = u / (PPW + 1);
        c = 2 * K * (u - r * (PPW + 1));
        if constexpr (D == 3) {
          j2 = 1 + r / m;
          j1 = 1 + (r - (r / m) * m);
        } else {
          j1 = 1 + r;
        }
      }
      if (c < seg) xw.store(0, (unsigned)((D == 3 ? j2 * n1d2 : 0) + j1 * n1d + c) * (unsigned)sizeof(T), T(0));
    }
  }
  // the lane's reciprocal eigenvalue sums: fetched with the first loads where the registers allow it
  constexpr bool kEarly = RC * m * sizeof(T) <= 104;
  auto fetch_inv = [&]() {
    const DevTables<T>& tb = tab_fresh<T>(K);
#pragma unroll
    for (int rr = 0; rr < RC; ++rr) {
      const int t = rr * NT + tid, r = D == 3 ? t - div_small<mm>(t) * mm : t - div_small<m>(t) * m;
#pragma unroll
      for (int a = 0; a < m; ++a) iv[rr][a] = D == 3 ? tb.inv3[r * m + a] : tb.inv2[r * m + a];
    }
  };
  if constexpr (kEarly) fetch_inv();
  // ---- S^T along the slowest axis
#pragma unroll
  for (int rr = 0; rr < RC; ++rr) {
    int q, i1, i0;
    unsigned off;
    if (line(rr * NT + tid, q, i1, i0, off)) {
      T r[m];
      apply_st<T, K>(v[rr], r);
      const int o = lds_base(D == 3 ? i1 * L::SI1 + q * mm + i0 : i0 * L::T0 + q * m);
#pragma unroll
      for (int a = 0; a < m; ++a) smem[o + a * (D == 3 ? m : 1)] = r[a];
    }
  }
  __syncthreads();
  if constexpr (D == 3) {
    // ---- S^T along x1: lines (q, a2, i0)
    T* W5 = smem + L::A;
#pragma unroll
    for (int rr = 0; rr < RC; ++rr) {
      const int t = rr * NT + tid;
      if (t < NB) {
        T in[m], r[m];
#pragma unroll
        for (int i = 0; i < m; ++i) in[i] = smem[i * L::SI1 + t];
        apply_st<T, K>(in, r);
        const int g = div_small<m>(t), i0 = t - g * m;
        const int o = lds_base(i0 * L::SI0 + g * m);
#pragma unroll
        for (int a = 0; a < m; ++a) W5[o + a] = r[a];
      }
    }
    __syncthreads();
  }
  // ---- S^T along x0, 1 / (sum of eigenvalues), S along x0: lines (q, a2, a1) / (q, a1)
  if constexpr (!kEarly) fetch_inv();
  {
    const T* in0 = D == 3 ? smem + L::A : smem;
    T* out0 = D == 3 ? smem : smem + L::A;
#pragma unroll
    for (int rr = 0; rr < RC; ++rr) {
      const int t = rr * NT + tid;
      if (t < NB) {
        T in[m], z[m], w[m];
#pragma unroll
        for (int i = 0; i < m; ++i) in[i] = in0[i * (D == 3 ? L::SI0 : L::T0) + t];
        apply_st<T, K>(in, z);
#pragma unroll
        for (int a = 0; a < m; ++a) z[a] *= iv[rr][a];
        apply_s<T, K>(z, w);
        int o;
        if constexpr (D == 3) {
          const int q = div_small<mm>(t), r = t - q * mm, a2 = div_small<m>(r), a1 = r - a2 * m;
          o = lds_base(a1 * L::SA1 + q * mm + a2 * m);
        } else {
          const int q = div_small<m>(t), a1 = t - q * m;
          o = lds_base(a1 * L::T0 + q * m);
        }
#pragma unroll
        for (int i = 0; i < m; ++i) out0[o + i] = w[i];
      }
    }
  }
  __syncthreads();
  if constexpr (D == 3) {
    // ---- S along x1: lines (q, a2, i0)
    T* W7 = smem + L::A;
#pragma unroll
    for (int rr = 0; rr < RC; ++rr) {
      const int t = rr * NT + tid;
      if (t < NB) {
        T in[m], w[m];
#pragma unroll
        for (int a = 0; a < m; ++a) in[a] = smem[a * L::SA1 + t];
        apply_s<T, K>(in, w);
        const int q = div_small<mm>(t), r = t - q * mm, a2 = div_small<m>(r), i0 = r - a2 * m;
        const int o = lds_base(a2 * L::SA2 + q * m + i0);
#pragma unroll
        for (int i = 0; i < m; ++i) W7[o + i * (PPW * m)] = w[i];
      }
    }
    __syncthreads();
  }
  // ---- S along the slowest axis, straight to global
#pragma unroll
  for (int rr = 0; rr < RC; ++rr) {
    const int t = rr * NT + tid;
    int q, i1, i0;
    unsigned off;
    if (line(t, q, i1, i0, off)) {
      T in[m], w[m];
#pragma unroll
      for (int a = 0; a < m; ++a) in[a] = smem[L::A + a * (D == 3 ? L::SA2 : L::T0) + t];
      apply_s<T, K>(in, w);
#pragma unroll
      for (int i = 0; i < m; ++i) xw.store(pl[i], off, ZERO ? sol_scale * w[i] : fma(sol_scale, w[i], xo[rr][i]));
    }
  }
}

// Launch shapes of these passes, as EigShapes (no shared layout): the fastest of 4-6 per row.  Measured, additive step
// per pass, us, against the closure-free lines form they replace (one node line order, two patches per workgroup in 3D
// Q4): 3D degree 4 64^3 cells FP32 29.4 (39.3), FP64 56.3 (59.9); degree 3 64^3 FP32 12.7 (21.2); degree 5 32^3 FP32
// 9.9 (14.1); first colour from zero, 3D Q4 64^3 FP32 26.8.
template <int D, int K, typename T>
struct AddShapes {
  static constexpr int PPW = D == 3 ? (K == 1 ? 64 : K == 2 ? 16 : K == 3 ? 8 : K == 4 ? 4 : K <= 6 ? 2 : 1)
                                    : (K == 1 ? 64 : K == 2 ? 42 : K == 3 ? 12 : K == 4 ? 16 : K == 5 ? 7 : K == 6 ? 5 : 4);
  static constexpr int NT = D == 3 ? (K == 1 ? 64 : K == 2 || K == 5 ? 192 : 256) : (K == 2 || K == 4 ? 128 : 64);
  using Large = EigShape<PPW, NT, false>;
  using Small = EigShape<(D == 3 ? (K == 1 ? 16 : K == 2 ? 4 : K == 3 ? 2 : 1) : (K == 1 ? 16 : K <= 4 ? 8 : 4)),
                         (D == 3 ? (K <= 3 ? 64 : K == 7 ? 192 : 128) : 64), false>;
};

// ------------------------------------------------------------------ several colours in one launch
//
// Small levels are bound by launches: a pass takes 2.5-3 us from one kernel's end to the next one's start and
// 1-2 us of work.  The colours that differ in the parity of x0 only (c and c ^ 1) touch a row of patches along
// x0 independently of all other rows: the closures of a row's patches span the same x1 and x2 range, and the
// nodes that the two colours update lie strictly inside it.  So one workgroup can run both colours of a row, one
// after the other, without any synchronisation between workgroups; likewise four colours (x0 and x1 parities) of
// a layer of patches in 3D, and all colours of the whole grid.  Span 1, 2, 3: row, layer, grid (2D: 1 row,
// 2 grid).  The workgroup's teams of threads take the row's (layer's, grid's) blocks of patches in turn.
// A pass here is the eigenbasis form without a look at old interior values, so it serves corrections; ADD: the
// additive pass.
template <int D, int K, typename T>
struct FusedTeams;  // SH: a team's shape; N: teams per workgroup
template <typename T> struct FusedTeams<3, 1, T> { using SH = Q1Shape<64>; static constexpr int N = 8; };
template <typename T> struct FusedTeams<3, 2, T> { using SH = EigShape<4, 128, false>; static constexpr int N = 4; };
template <typename T> struct FusedTeams<3, 3, T> { using SH = EigShape<2, 128, false>; static constexpr int N = 4; };
template <typename T> struct FusedTeams<3, 4, T> { using SH = EigShape<2, 128, false>; static constexpr int N = 4; };
template <typename T> struct FusedTeams<3, 5, T> { using SH = EigShape<1, 128, false>; static constexpr int N = 4; };
template <typename T> struct FusedTeams<3, 6, T> { using SH = EigShape<1, 192, true>; static constexpr int N = 4; };
template <typename T> struct FusedTeams<3, 7, T> { using SH = EigShape<1, 256, true>; static constexpr int N = 4; };
template <typename T> struct FusedTeams<2, 1, T> { using SH = Q1Shape<64>; static constexpr int N = 8; };
template <typename T> struct FusedTeams<2, 2, T> { using SH = EigShape<8, 64, false>; static constexpr int N = 8; };
template <typename T> struct FusedTeams<2, 3, T> { using SH = EigShape<4, 64, false>; static constexpr int N = 8; };
template <typename T> struct FusedTeams<2, 4, T> { using SH = EigShape<4, 128, false>; static constexpr int N = 8; };
template <typename T> struct FusedTeams<2, 5, T> { using SH = EigShape<4, 128, false>; static constexpr int N = 8; };
template <typename T> struct FusedTeams<2, 6, T> { using SH = EigShape<4, 128, false>; static constexpr int N = 8; };
template <typename T> struct FusedTeams<2, 7, T> { using SH = EigShape<4, 128, false>; static constexpr int N = 8; };

struct FusedMembers {
  const void* b[kMaxGroup];
  void* x[kMaxGroup];
};

// LDS of a team's pass (T words).
template <int D, int K, typename SH, bool ADD>
constexpr int team_lds() {
  if constexpr (ADD) return (AddLds<D, K, SH>::total + 3) & ~3;
  else if constexpr (K == 1) return 0;
  else if constexpr (D == 3) return (EigLds3<K, SH>::total + 3) & ~3;
  else return (EigLds2<K, SH>::total + 3) & ~3;
}
template <int D, int K, typename T, bool ADD>
__global__ __launch_bounds__((FusedTeams<D, K, T>::SH::NT * FusedTeams<D, K, T>::N)) void colour_span_kernel(
    FusedMembers mem, long long n1d, int half, int span, int first, int n_colours, int step, int clear, T res_scale,
    T sol_scale) {
  using SH = typename FusedTeams<D, K, T>::SH;
  constexpr int TEAMS = FusedTeams<D, K, T>::N, NT = SH::NT, PPW = SH::PPW;
  constexpr int kLds = team_lds<D, K, SH, ADD>();
  __shared__ __align__(16) T smem[max_of(kLds * TEAMS, 1)];
  const int team = __builtin_amdgcn_readfirstlane((int)threadIdx.x / NT), tid = (int)threadIdx.x - team * NT;
  const T* b = (const T*)mem.b[blockIdx.y];
  T* x = (T*)mem.x[blockIdx.y];
  const int w = blockIdx.x;
  if (clear) {
    // x holds anything: 0 on the closures of this workgroup's row, layer or grid.  Neighbouring workgroups write
    // the same zeros on shared faces, and nobody updates those in this launch.
    const int cnt = half;  // colour 0: half patches per axis
    const long long nr1 = span == 1 ? 2 * K + 1 : n1d;
    const int t1 = span == 1 ? w % cnt : 0, t2 = span == 1 ? w / cnt : w;
    const long long o1 = span == 1 ? 2LL * K * t1 : 0;
    const long long nr2 = D == 2 ? 1 : span == 3 ? n1d : 2 * K + 1, o2 = D == 2 || span == 3 ? 0 : 2LL * K * t2;
    const long long rows = nr1 * nr2;
    const int len = (int)n1d;
    for (long long r = threadIdx.x >> 6; r < rows; r += blockDim.x >> 6) {
      const long long j2 = r / nr1, j1 = r - j2 * nr1;
      T* row = x + ((o2 + j2) * n1d * (D == 3 ? 1 : 0) + o1 + j1) * n1d;
      for (int i = threadIdx.x & 63; i < len; i += 64) row[i] = T(0);
    }
    __syncthreads();
  }
  for (int ci = 0; ci < n_colours; ++ci) {
    const int c = first + ci * step;
    const int p0 = c & 1, p1 = (c >> 1) & 1, p2 = (c >> 2) & 1;
    const int cnt0 = half - p0, cnt1 = half - p1, cnt2 = D == 3 ? half - p2 : 1;
    const int groups0 = (cnt0 + PPW - 1) / PPW;
    const int per = groups0 * (span >= 2 ? cnt1 : 1) * (span >= 3 ? cnt2 : 1);
    for (int base = 0; base < per; base += TEAMS) {
      const int k = base + team;
      const bool active = k < per;
      const unsigned blk = (unsigned)(w * per + (active ? k : 0));
      T* tm = smem + team * kLds;
      if constexpr (ADD)
        colour_pass_add<D, K, T, false, SH>(tm, b, x, n1d, p0, p1, p2, cnt0, cnt1, groups0, sol_scale, blk, tid, active);
      else if constexpr (K == 1)
        colour_pass_q1<D, T, true, PPW>(b, x, n1d, p0, p1, p2, cnt0, cnt1, groups0, res_scale, sol_scale, blk, tid,
                                        active);
      else if constexpr (D == 3)
        colour_pass_eig3<K, T, false, SH>(tm, b, x, n1d, p0, p1, p2, cnt0, cnt1, groups0, sol_scale, blk, tid, active);
      else
        colour_pass_eig2<K, T, false, SH>(tm, b, x, n1d, p0, p1, cnt0, cnt1, groups0, sol_scale, blk, tid, active);
      __syncthreads();
    }
  }
}

// Calls f.template operator()<D, K>() for the run-time (dim, degree).
template <typename F>
static hipError_t with_degree(int dim, int k, F f) {
  switch (dim * 10 + k) {
    case 21: return f(std::integral_constant<int, 2>{}, std::integral_constant<int, 1>{});
    case 22: return f(std::integral_constant<int, 2>{}, std::integral_constant<int, 2>{});
    case 23: return f(std::integral_constant<int, 2>{}, std::integral_constant<int, 3>{});
    case 24: return f(std::integral_constant<int, 2>{}, std::integral_constant<int, 4>{});
    case 25: return f(std::integral_constant<int, 2>{}, std::integral_constant<int, 5>{});
    case 26: return f(std::integral_constant<int, 2>{}, std::integral_constant<int, 6>{});
    case 27: return f(std::integral_constant<int, 2>{}, std::integral_constant<int, 7>{});
    case 31: return f(std::integral_constant<int, 3>{}, std::integral_constant<int, 1>{});
    case 32: return f(std::integral_constant<int, 3>{}, std::integral_constant<int, 2>{});
    case 33: return f(std::integral_constant<int, 3>{}, std::integral_constant<int, 3>{});
    case 34: return f(std::integral_constant<int, 3>{}, std::integral_constant<int, 4>{});
    case 35: return f(std::integral_constant<int, 3>{}, std::integral_constant<int, 5>{});
    case 36: return f(std::integral_constant<int, 3>{}, std::integral_constant<int, 6>{});
    case 37: return f(std::integral_constant<int, 3>{}, std::integral_constant<int, 7>{});
  }
  return hipErrorInvalidValue;
}

template <int D, int K, typename T, bool ADD>
static hipError_t smooth_fused(const LevelGeom& g, int span, bool reverse, bool clear, const ColourPassMember* mem, int nm,
                               hipStream_t st) {
  using FT = FusedTeams<D, K, T>;
  const int half = (int)(g.ncells / 2), top = D;  // span `top`: the whole grid
  const int colours = 1 << span, sets = (1 << D) / colours;
  const T res_scale = (T)(D == 3 ? g.h : 1.0), sol_scale = (T)(D == 3 ? 1.0 / g.h : 1.0);
  for (int i0 = 0; i0 < nm; i0 += kMaxGroup) {
    const int n = nm - i0 < kMaxGroup ? nm - i0 : kMaxGroup;
    FusedMembers fm{};
    for (int i = 0; i < n; ++i) {
      fm.b[i] = mem[i0 + i].b;
      fm.x[i] = mem[i0 + i].x;
    }
    for (int j = 0; j < sets; ++j) {
      const int set = reverse ? sets - 1 - j : j;
      const int first = set * colours + (reverse ? colours - 1 : 0);
      int units = 1;  // workgroups: rows, layers, or the grid
      for (int a = span; a < top; ++a) units *= half - ((first >> a) & 1);
      hipLaunchKernelGGL((colour_span_kernel<D, K, T, ADD>), dim3(units, n), dim3(FT::SH::NT * FT::N), 0, st, fm, g.n1d, half,
                         span, first, colours, reverse ? -1 : 1, clear && j == 0 ? 1 : 0, res_scale, sol_scale);
      hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
  }
  return hipSuccess;
}

// Fills this file's tables on the current device.
static hipError_t upload_tables() {
  static DevTables<double> h64[kMaxDegree + 1];
  static DevTables<float> h32[kMaxDegree + 1];
  for (int k = 1; k <= kMaxDegree; ++k) {
    fill_dev_tables(k, h64[k]);
    fill_dev_tables(k, h32[k]);
  }
  hipError_t e = hipMemcpyToSymbol(HIP_SYMBOL(g_tab64), h64, sizeof(h64));
  if (e != hipSuccess) return e;
  return hipMemcpyToSymbol(HIP_SYMBOL(g_tab32), h32, sizeof(h32));
}

}  // namespace vps
