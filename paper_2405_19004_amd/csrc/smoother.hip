// Vertex-patch smoother colour pass for gfx950 (the hot kernel).
//
// One launch processes every patch of one colour (Alg. 3: colours are
// sequential, patches inside a colour are disjoint and run in parallel).  Per
// patch j, multiplicative mode computes
//   r_j = b_j^I - Abar_j x_j          localised residual (Sec. 2.2)
//   x_j^I += A_j^{-1} r_j             fast diagonalisation (eq:inverse2d/3d)
// where Abar_j = sum_dir (x) of 1D patch matrices (eq:tensorproduct_2d/3d) is
// applied by sum factorisation with the partial products reused across
// directions (Sec. 3.1.1), and A_j^{-1} = (S x..x S)(sum Lambda)^{-1}(S x..x S)^T.
// Additive mode skips the residual: x^I += A_j^{-1} b_j^I.
// Boundary mode (Sec. 4.1.3, eq:A_ib_2d/3d) uses that the local solver is exact:
//   x_j^I <- A_j^{-1} (b_j^I - A^{IB} x_j^B),
// i.e. the residual is formed with the patch interior taken as zero and the
// interior is overwritten, so x^I is never loaded.
// The multiplicative pass has two forms: the eigenbasis form, which works on the boundary nodes of the
// closures only, and the residual form as written above; kernels.hpp says which serves what.
//
// Mapping (designed for CDNA4, not a translation of the paper's CUDA):
//  * a workgroup owns PPW patches that are consecutive along x0 inside the
//    colour; their closures tile one contiguous x0 segment of 2k*PPW+1 nodes,
//    so the closure load is one coalesced sweep over rows and shared faces are
//    read once;
//  * every 1D contraction is done by a thread that holds one whole line (a
//    1D fibre of the patch tensor) in registers and multiplies it by the 1D
//    matrix, whose entries are wave-uniform and come from constant memory
//    through the scalar cache (SGPR operands of v_fma);
//  * LDS only transposes between directions: one write and one read per value
//    per direction change, never one LDS read per multiply-add.
// No atomics: patches of one colour write disjoint interiors.
#include "device_common.hpp"
#include "kernels.hpp"
#include "patch_tables_gen.hpp"

#include <cmath>
#include <type_traits>
#include <vector>

namespace vps {

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

// ------------------------------------------------------------------ residual form

// LDS of the 3D multiplicative pass below (T words).  Buffer A holds PM, PA [i2][j1][c], later the
// results of stages C and E; buffer B holds U, V, later those of D and F.  Every transpose buffer
// after PM/PA is laid out [loop index of the reading stage][reading task], the outer stride padded
// (mod 32) so that the writing lanes also touch distinct banks: for U, V and the D->E buffer the
// residue was searched per degree with a bank model of both sides (4- and 8-byte words); the others
// are distinct by construction.
template <int K, int PPW>
struct Mult3Lds {
  static constexpr int n = 2 * K + 1, m = 2 * K - 1, mm = m * m;
  static constexpr int RS = 2 * K * PPW + 1;  // closure columns of the workgroup along x0
  static constexpr int PM = m * n * RS;       // one of PM, PA
  static constexpr int kSURes[8] = {0, 11, 7, 19, 15, 27, 23, 3};
  static constexpr int SU = pad32(PPW * mm, kSURes[K]);  // U, V  [j1][q][i2][i0]
  static constexpr int SW = pad32(PPW * mm, m);          // C->D  [i2][q][a1][i0]
  static constexpr int kSW2Res[8] = {0, 0, 3, 13, 23, 25, 3, 5};
  static constexpr int SW2 = pad32(PPW * mm, kSW2Res[K]); // D->E  [i0][q][a2][a1]
  static constexpr int SW3 = pad32(PPW * mm, 1);         // E->F  [a1][q][a2][i0]
  static constexpr int SW4 = pad32(PPW * mm, m);         // F->G  [a2][q][i1][i0]
  static constexpr int max3(int a, int b, int c) { return a > b ? (a > c ? a : c) : (b > c ? b : c); }
  static constexpr int A = max3(2 * PM, m * SW, m * SW3);
  static constexpr int B = max3(2 * n * SU, m * SW2, m * SW4);
  // Aliased layout: PM/PA, U/V and the C->D buffer all start at word 0 (stages B and C compute
  // every line, the workgroup synchronises, then they write over their inputs); the D->E and F->G
  // buffers follow the larger of C->D and E->F, which starts at 0 again.  Measured 11-45% faster for
  // degrees 2-7 (occupancy: 3D Q4 goes from 33 to 17 KB of LDS, from 8 to 18 waves per compute unit).
  static constexpr bool AL = K >= 2;
  static constexpr int X1 = m * SW > m * SW3 ? m * SW : m * SW3;
  static constexpr int ALT = max3(2 * PM, 2 * n * SU, X1 + (m * SW2 > m * SW4 ? m * SW2 : m * SW4));
  static constexpr int total = AL ? ALT : A + B;
  static constexpr int offP = 0, offUV = AL ? 0 : A;
  static constexpr int offW = 0, offW2 = AL ? X1 : A, offW3 = 0, offW4 = AL ? X1 : A;
};

// 3D multiplicative colour pass, closure contracted along x2 first.  Every thread of stage A loads
// one closure column along x2 straight from global memory and contracts it in registers, so the
// closure itself never goes through LDS.  Stages (lines, the axis contracted):
//   A  columns (j1, c)    x2: PM = M2 x, PA = A2 x                         -> A [i2][j1][c]
//   B  lines (q, i2, j1)  x0: U = M0 PM, V = A0 PM + M0 PA                  -> B [j1][q][i2][i0]
//   C  lines (q, i2, i0)  x1: r = b - h (A1 U + M1 V), then S^T along x1    -> A [i2][q][a1][i0]
//   D  lines (q, a1, i0)  S^T along x2                                      -> B [i0][q][a2][a1]
//   E  lines (q, a2, a1)  S^T along x0, 1/(lam2 + lam1 + lam0), S along x0  -> A [a1][q][a2][i0]
//   F  lines (q, a2, i0)  S along x1                                        -> B [a2][q][i1][i0]
//   G  lines (q, i1, i0)  S along x2, x^I += correction / h
// The three terms of the patch operator are those of the other contraction order up to rounding
// (1D factors on different axes commute).  b is read on the x1 lines of stage C; the update runs on
// the x2 lines of stage G, whose lanes share one node plane per access, and takes the old x^I from
// the thread's own stage A column.
template <int K, typename T, int PPW>
__device__ __forceinline__ void colour_pass_mult3(T* __restrict__ smem, const T* __restrict__ b, T* __restrict__ x,
                                                  long long n1d, int p0, int p1, int p2, int cnt0, int cnt1,
                                                  int groups0, T res_scale, T sol_scale, unsigned blk) {
  constexpr int n = 2 * K + 1, m = 2 * K - 1, mm = m * m;
  constexpr int NT = SmootherShape<3, K>::NT;
  using PT = gen::PatchTables<T, K>;
  using L = Mult3Lds<K, PPW>;
  constexpr int RS = L::RS;

  const ColourBlock cb = colour_block<3, K, PPW>(blk, p0, p1, p2, cnt0, cnt1, groups0);
  const int P = cb.count;
  const long long s0 = cb.s0, s1 = cb.s1, s2 = cb.s2;
  const long long n1d2 = n1d * n1d;
  const int tid = threadIdx.x;
  const int seg = 2 * K * P + 1;  // valid closure columns along x0
  // byte offsets inside the workgroup's closure fit in 32 bits (checked by the launcher)
  const int ld1 = (int)n1d;
  T* xo = x + (s2 * n1d2 + s1 * n1d + s0);  // closure corner of the first patch
  const T* bo = b + (s2 * n1d2 + s1 * n1d + s0);

  // b on the x1 lines (q, i2, i0) of stage C, prefetched now (tasks past the last patch are clamped
  // to it, so every load is in bounds); xpre is filled by stage A
  constexpr int NB = PPW * mm;
  constexpr int RB = (NB + NT - 1) / NT;
  T bpre[RB][m], xpre[RB][m];
  unsigned xoff[RB];  // byte offset of node (0, 1 + i1, 1 + i0) of stage G's line from the corner
#pragma unroll
  for (int rr = 0; rr < RB; ++rr) {
    const int task = rr * NT + tid;
    int q = task / mm;
    const int r = task - q * mm;
    const int hi = r / m, lo = r - hi * m;  // (i2, i0) for stage C, (i1, i0) for stage G
    q = min(q, P - 1);
    const unsigned boff = (unsigned)(((1 + hi) * n1d2 + 2 * K * q + 1 + lo) * (long long)sizeof(T));
    xoff[rr] = (unsigned)(((1 + hi) * n1d + 2 * K * q + 1 + lo) * (long long)sizeof(T));
#pragma unroll
    for (int i = 0; i < m; ++i) bpre[rr][i] = ld_lane(bo + (1 + i) * ld1, boff);
  }

  // ---- A: closure columns along x2 -> PM, PA.  Tasks 0 .. NB-1 are the patch-interior columns in
  //      the order of stage G's lines (q, i1, i0), so a thread keeps the old x^I of its stage G line
  //      from its own column; the face columns (j1 on the closure boundary, or c on a patch
  //      boundary) follow.  Dirichlet nodes count as 0 (the boundary entries of x are not read as
  //      values).
  {
    T* PM = smem + L::offP;
    T* PA = PM + L::PM;
    constexpr int NF = 2 * RS + (n - 2) * (PPW + 1);  // face columns
    constexpr int NA = NB + NF;
    const bool lo0 = s0 == 0, hi0 = s0 + seg - 1 == n1d - 1;
    const bool lo1 = s1 == 0, hi1 = s1 + n - 1 == n1d - 1;
    const bool lo2 = s2 == 0, hi2 = s2 + n - 1 == n1d - 1;
#pragma unroll
    for (int it = 0; it < (NA + NT - 1) / NT; ++it) {
      const int t = it * NT + tid;
      int j1, c;
      if (t < NB) {
        const int q = t / mm, r = t - q * mm, i1 = r / m;
        j1 = 1 + i1;
        c = 2 * K * q + 1 + (r - i1 * m);
      } else {
        const int f = t - NB;
        if (f < 2 * RS) {
          j1 = f < RS ? 0 : n - 1;
          c = f < RS ? f : f - RS;
        } else {
          const int g = f - 2 * RS, jj = g / (PPW + 1);
          j1 = 1 + jj;
          c = 2 * K * (g - jj * (PPW + 1));
        }
      }
      if (t < NA && c < seg) {
        const unsigned off = (unsigned)(j1 * ld1 + c) * (unsigned)sizeof(T);
        T v[n];
#pragma unroll
        for (int j = 0; j < n; ++j) v[j] = ld_lane(xo + j * n1d2, off);
        if (it < RB && t < NB) {  // patch-interior column: never a Dirichlet node
#pragma unroll
          for (int i = 0; i < m; ++i) xpre[it < RB ? it : 0][i] = v[1 + i];
        }
        const bool zc = (c == 0 && lo0) || (c == seg - 1 && hi0) || (j1 == 0 && lo1) || (j1 == n - 1 && hi1);
        if (zc) {
#pragma unroll
          for (int j = 0; j < n; ++j) v[j] = T(0);
        }
        if (lo2) v[0] = T(0);
        if (hi2) v[n - 1] = T(0);
        const int o = lds_base(j1 * RS + c);
#pragma unroll
        for (int i = 0; i < m; ++i) {
          T sm = T(0), sa = T(0);
#pragma unroll
          for (int j = 0; j < n; ++j) {
            sm = fma_tab(PT::Mc[i * n + j], v[j], sm);
            sa = fma_tab(PT::Ac[i * n + j], v[j], sa);
          }
          PM[o + i * n * RS] = sm;
          PA[o + i * n * RS] = sa;
        }
      }
    }
  }
  __syncthreads();
  // ---- B: x0 lines (q, i2, j1), j1 fastest -> U, V
  {
    const T* PM = smem + L::offP;
    const T* PA = PM + L::PM;
    T* U = smem + L::offUV;
    T* V = U + n * L::SU;
    // x0 line of a task: U and V rows into su, sv; false past the workgroup's patches
    auto line = [&](int task, T* su, T* sv) -> bool {
      const int q = task / (m * n), r = task - q * (m * n);
      const int i2 = r / n, j1 = r - i2 * n;
      if (task >= PPW * m * n || q >= P) return false;
      const int ri = lds_base((i2 * n + j1) * RS + 2 * K * q);
      T pm[n], pa[n];
#pragma unroll
      for (int c = 0; c < n; ++c) {
        pm[c] = PM[ri + c];
        pa[c] = PA[ri + c];
      }
#pragma unroll
      for (int i = 0; i < m; ++i) {
        T au = T(0), av = T(0);
#pragma unroll
        for (int c = 0; c < n; ++c) {
          au = fma_tab(PT::Mc[i * n + c], pm[c], au);
          av = fma_tab(PT::Ac[i * n + c], pm[c], av);
          av = fma_tab(PT::Mc[i * n + c], pa[c], av);
        }
        su[i] = au;
        sv[i] = av;
      }
      return true;
    };
    auto put = [&](int task, const T* su, const T* sv) {
      const int q = task / (m * n), r = task - q * (m * n);
      const int i2 = r / n, j1 = r - i2 * n;
      const int o = lds_base(j1 * L::SU + (q * m + i2) * m);
#pragma unroll
      for (int i = 0; i < m; ++i) {
        U[o + i] = su[i];
        V[o + i] = sv[i];
      }
    };
    if constexpr (L::AL) {
      // U/V overwrite PM/PA: every line first, then the writes
      constexpr int RB2 = (PPW * m * n + NT - 1) / NT;
      T su[RB2][m], sv[RB2][m];
      bool ok[RB2];
#pragma unroll
      for (int rr = 0; rr < RB2; ++rr) ok[rr] = line(rr * NT + tid, su[rr], sv[rr]);
      __syncthreads();
#pragma unroll
      for (int rr = 0; rr < RB2; ++rr)
        if (ok[rr]) put(rr * NT + tid, su[rr], sv[rr]);
    } else {
      for (int base = 0; base < PPW * m * n; base += NT) {
        T su[m], sv[m];
        if (line(base + tid, su, sv)) put(base + tid, su, sv);
      }
    }
  }
  __syncthreads();
  // ---- C: x1 lines (q, i2, i0): residual, then S^T along x1.  Aliased layout: the C->D buffer
  //      overwrites U/V, so every line is computed before the workgroup synchronises and writes.
  T tc[RB][m];
#pragma unroll
  for (int rr = 0; rr < RB; ++rr) {
    const int task = rr * NT + tid;
    const int q = task / mm;
    if (task < NB && q < P) {
      const T* U = smem + L::offUV;
      const T* V = U + n * L::SU;
      T u[n], v[n];
#pragma unroll
      for (int j = 0; j < n; ++j) {
        u[j] = U[j * L::SU + task];
        v[j] = V[j * L::SU + task];
      }
      T res[m];
#pragma unroll
      for (int i = 0; i < m; ++i) {
        T sres = T(0);
#pragma unroll
        for (int j = 0; j < n; ++j) {
          sres = fma_tab(PT::Ac[i * n + j], u[j], sres);
          sres = fma_tab(PT::Mc[i * n + j], v[j], sres);
        }
        res[i] = fma(-res_scale, sres, bpre[rr][i]);
      }
      apply_st<T, K>(res, tc[rr]);
    }
  }
  if constexpr (L::AL) __syncthreads();
  {
    T* W = smem + L::offW;
#pragma unroll
    for (int rr = 0; rr < RB; ++rr) {
      const int task = rr * NT + tid;
      const int q = task / mm;
      if (task < NB && q < P) {
        const int r = task - q * mm, i2 = r / m, i0 = r - i2 * m;
        const int o = lds_base(i2 * L::SW + q * mm + i0);
#pragma unroll
        for (int a = 0; a < m; ++a) W[o + a * m] = tc[rr][a];
      }
    }
  }
  __syncthreads();
  // ---- D: x2 lines (q, a1, i0): S^T along x2
  for (int base = 0; base < PPW * mm; base += NT) {
    const int task = base + tid;
    const int q = task / mm;
    if (task < PPW * mm && q < P) {
      const T* W = smem + L::offW;
      T* W2 = smem + L::offW2;
      const int r = task - q * mm, a1 = r / m, i0 = r - a1 * m;
      T in[m];
#pragma unroll
      for (int i = 0; i < m; ++i) in[i] = W[i * L::SW + task];
      T t[m];
      apply_st<T, K>(in, t);
      const int o = lds_base(i0 * L::SW2 + q * mm + a1);
#pragma unroll
      for (int a = 0; a < m; ++a) W2[o + a * m] = t[a];
    }
  }
  __syncthreads();
  // ---- E: x0 lines (q, a2, a1): S^T along x0, eigenvalue scaling, S along x0
  for (int base = 0; base < PPW * mm; base += NT) {
    const int task = base + tid;
    const int q = task / mm;
    if (task < PPW * mm && q < P) {
      const T* W2 = smem + L::offW2;
      T* W3 = smem + L::offW3;
      const DevTables<T>& tb = tab_fresh<T>(K);
      const int r = task - q * mm, a2 = r / m, a1 = r - a2 * m;
      T in[m], z[m];
#pragma unroll
      for (int i = 0; i < m; ++i) in[i] = W2[i * L::SW2 + task];
      apply_st<T, K>(in, z);
#pragma unroll
      for (int a = 0; a < m; ++a) z[a] *= tb.inv3[r * m + a];
      T w[m];
      apply_s<T, K>(z, w);
      const int o = lds_base(a1 * L::SW3 + q * mm + a2 * m);
#pragma unroll
      for (int i = 0; i < m; ++i) W3[o + i] = w[i];
    }
  }
  __syncthreads();
  // ---- F: x1 lines (q, a2, i0): S along x1
  for (int base = 0; base < PPW * mm; base += NT) {
    const int task = base + tid;
    const int q = task / mm;
    if (task < PPW * mm && q < P) {
      const T* W3 = smem + L::offW3;
      T* W4 = smem + L::offW4;
      const int r = task - q * mm, a2 = r / m, i0 = r - a2 * m;
      T in[m];
#pragma unroll
      for (int a = 0; a < m; ++a) in[a] = W3[a * L::SW3 + task];
      T w[m];
      apply_s<T, K>(in, w);
      const int o = lds_base(a2 * L::SW4 + q * mm + i0);
#pragma unroll
      for (int i = 0; i < m; ++i) W4[o + i * m] = w[i];
    }
  }
  __syncthreads();
  // ---- G: x2 lines (q, i1, i0): S along x2 and x^I += correction, straight to global
#pragma unroll
  for (int rr = 0; rr < RB; ++rr) {
    const int task = rr * NT + tid;
    const int q = task / mm;
    if (task < NB && q < P) {
      const T* W4 = smem + L::offW4;
      T in[m];
#pragma unroll
      for (int a = 0; a < m; ++a) in[a] = W4[a * L::SW4 + task];
      T w[m];
      apply_s<T, K>(in, w);
#pragma unroll
      for (int i = 0; i < m; ++i) st_lane(xo + (1 + i) * n1d2, xoff[rr], fma(sol_scale, w[i], xpre[rr][i]));
    }
  }
}

// Wide shape of the 3D Q4 FP32 colour pass (residual form): five patches per workgroup on 256 threads.  Its 49-line stages fill 245 of 256 lanes,
// against 98 of 128 for the two-patch default, which cuts the vector instructions per patch by
// about a fifth.  A row of patches along x0 that is not a multiple of five leaves a partial
// workgroup, so launches take it only on long rows (at most kWideIdle idle patch slots per row, as a
// fraction of the row).
constexpr int kWidePPW = 5, kWideNT = 256;
constexpr double kWideIdle = 0.15;
template <int D, int K, typename T, int MODE>
struct HasWideForm {
  static constexpr bool value = D == 3 && K == 4 && sizeof(T) == 4 &&
                                MODE == kModeResidual;
};
template <int D, int K, typename T, int MODE, int PPW>
struct IsWide {
  static constexpr bool value = HasWideForm<D, K, T, MODE>::value && PPW == kWidePPW;
};

// Degrees whose default 3D residual-form shape also takes the paired layout (the wide
// shape always does): 1-2.5% faster for degrees 5-7 (3D Q7: 30.8 -> 24.8 KB), equal for 3 and 4.
template <int D, int K, typename T, int MODE, int PPW>
struct LinesPair {
  static constexpr bool value =
      IsWide<D, K, T, MODE, PPW>::value ||
      (D == 3 && MODE == kModeResidual && K >= 5 && PPW == SmootherShape<3, K>::PPW);
};

// The aliased LDS layout serves the default shape of the residual form where the shape asks for it (2D:
// always), and the wide shape.
template <int D, int K, typename T, int MODE, int PPW>
struct LinesAlias {
  static constexpr bool value =
      (D == 3 && MODE == kModeResidual && SmootherShape<3, K>::ALIAS && PPW == SmootherShape<3, K>::PPW) ||
      (D == 2 && MODE == kModeResidual && PPW == SmootherShape<2, K>::PPW) ||
      IsWide<D, K, T, MODE, PPW>::value;
};

// One workgroup's share of a colour pass: patches of block `blk` of the colour described by
// (p0, p1, p2, cnt0, cnt1, groups0) on a level with n1d nodes per direction.
template <int D, int K, typename T, int MODE, int PPW>
__device__ __forceinline__ void colour_pass_lines(T* __restrict__ smem, const T* __restrict__ b, T* __restrict__ x,
                                                  long long n1d, int p0, int p1, int p2, int cnt0, int cnt1,
                                                  int groups0, T res_scale, T sol_scale, unsigned blk) {
  constexpr int n = 2 * K + 1, m = 2 * K - 1, mm = m * m;
  constexpr int NT = IsWide<D, K, T, MODE, PPW>::value ? kWideNT : SmootherShape<D, K>::NT;
  // patch matrices and eigenvectors as compile-time constants (instruction literals / SGPR moves)
  using PT = gen::PatchTables<T, K>;
  using L = SmootherLds<D, K, T, PPW, LinesAlias<D, K, T, MODE, PPW>::value, LinesPair<D, K, T, MODE, PPW>::value>;
  constexpr int RS = L::RS;
  (void)p2;

  const ColourBlock cb = colour_block<D, K, PPW>(blk, p0, p1, p2, cnt0, cnt1, groups0);
  const int P = cb.count;
  const long long s0 = cb.s0, s1 = cb.s1, s2 = cb.s2;
  const long long n1d2 = n1d * n1d;
  const int tid = threadIdx.x;
  const int seg = 2 * K * P + 1;  // valid length of the closure row segment

  // Offsets inside one workgroup's block fit in 32 bits (checked by the launcher).
  const int ld1 = (int)n1d, ld2 = D == 3 ? (int)n1d2 : 0;
  const long long origin = (D == 3 ? s2 * n1d2 : 0) + s1 * n1d + s0;  // closure corner of the first patch
  T* xo = x + origin;  // same restrict object as x
  const T* bo = b + origin;

  // Lines along the slowest axis, task = (q, i1, i0) in 3D / (q, i0) in 2D with i0 fastest:
  // the residual stage reads b on them and the last stage updates x^I on them.  b is
  // prefetched now (clamped to a valid patch so the loads are always in bounds); the old x^I
  // comes from the closure in LDS.
  constexpr int NB = D == 3 ? PPW * mm : PPW * m;
  constexpr int RB = (NB + NT - 1) / NT;
  T bpre[RB][m], xpre[RB][m];
  unsigned loff[RB];  // byte offset of the line's first node from its plane
  int xoff[RB];
#pragma unroll
  for (int rr = 0; rr < RB; ++rr) {
    const int task = rr * NT + tid;
    int q, i1 = 0, i0;
    if constexpr (D == 3) {
      q = task / mm;
      const int r = task - q * mm;
      i1 = r / m;
      i0 = r - i1 * m;
    } else {
      q = task / m;
      i0 = task - q * m;
    }
    q = min(q, P - 1);
    // node (1 + i1, 1 + i0) of the patch's first interior plane, relative to that plane
    const int off = (D == 3 ? (1 + i1) * ld1 : 0) + 2 * K * q + 1 + i0;
    loff[rr] = (unsigned)off * (unsigned)sizeof(T);
    xoff[rr] = (D == 3 ? (n + 1 + i1) * RS : RS) + 2 * K * q + 1 + i0;  // node (i=0) in the LDS closure
    const int st = D == 3 ? ld2 : ld1;
#pragma unroll
    for (int i = 0; i < m; ++i) bpre[rr][i] = ld_lane(bo + st + i * st, loff[rr]);
  }

  // ---- closure segment -> LDS X [j2][j1][c].  Work item = (column c, row j1 in 3D); the
  // slowest axis is walked unrolled.  Every closure node lies inside the grid: loads are
  // unconditional and Dirichlet nodes are replaced by 0 (boundary entries of x are ignored).
  {
    T* X = smem + (D == 3 ? L::offX : L::offX2);
    constexpr int NW = D == 3 ? RS * n : RS;
    const bool lo1 = s1 == 0, hi1 = s1 + n - 1 == n1d - 1;
    const bool lo2 = D == 3 && s2 == 0, hi2 = D == 3 && s2 + n - 1 == n1d - 1;
    for (int w = tid; w < NW; w += NT) {
      const int c = w % RS, j1 = D == 3 ? w / RS : 0;
      const int cl = min(c, seg - 1);
      const long long gc = s0 + cl;
      bool bad = gc == 0 || gc == n1d - 1;
      if constexpr (D == 3) bad = bad || (j1 == 0 && lo1) || (j1 == n - 1 && hi1);
      const unsigned base = ((D == 3 ? j1 * ld1 : 0) + cl) * (unsigned)sizeof(T);
      const int sstride = D == 3 ? ld2 : ld1;
      T v[n];
#pragma unroll
      for (int j = 0; j < n; ++j) v[j] = ld_lane(xo + j * sstride, base);
      const bool lo = D == 3 ? lo2 : lo1, hi = D == 3 ? hi2 : hi1;
      if (c < seg) {
#pragma unroll
        for (int j = 0; j < n; ++j) {
          const bool zero = bad || (j == 0 && lo) || (j == n - 1 && hi);
          X[(D == 3 ? j * n + j1 : j) * RS + c] = zero ? T(0) : v[j];
        }
      }
    }
    __syncthreads();
    // old x^I of this thread's lines: patch-interior nodes are never Dirichlet nodes
#pragma unroll
    for (int rr = 0; rr < RB; ++rr) {
#pragma unroll
      for (int i = 0; i < m; ++i) xpre[rr][i] = X[xoff[rr] + i * (D == 3 ? n * RS : RS)];
    }
  }

  if constexpr (D == 3) {
    constexpr int SJ1 = L::SJ1, SJ2 = L::SJ2, SI1 = L::SI1, SI0 = L::SI0, SA1 = L::SA1, SA2 = L::SA2;
    {
      const T* X = smem + L::offX;
      T* PM = smem + L::offP;  // [j1][q][j2][i0]
      T* PA = PM + n * SJ1;
      using T2 = typename Pair<T>::type;
      T2* PP = reinterpret_cast<T2*>(smem + L::offP);  // paired layout: [j1][q][j2][i0]{M, A}
      constexpr int SJP2 = L::SJP / 2;                  // pair stride
      // ---- contract x0 with Mc and Ac: lines (q, j2, j1), j1 fastest
      if constexpr (L::AL) {
        // aliased: every line of the workgroup is read and contracted, then PM/PA overwrite X
        constexpr int NA = PPW * n * n, RA = (NA + NT - 1) / NT;
        T om[RA][m], oa[RA][m];
#pragma unroll
        for (int rr = 0; rr < RA; ++rr) {
          const int task = rr * NT + tid;
          const int q = task / (n * n), r = task - q * (n * n);
          const int j2 = r / n, j1 = r - j2 * n;
          if (task < NA && q < P) {
            T in[n];
            const int row = lds_base((j2 * n + j1) * RS + 2 * K * q);
#pragma unroll
            for (int j = 0; j < n; ++j) in[j] = X[row + j];
#pragma unroll
            for (int i = 0; i < m; ++i) {
              T sm = T(0), sa = T(0);
#pragma unroll
              for (int j = 0; j < n; ++j) {
                sm = fma_tab(PT::Mc[i * n + j], in[j], sm);
                sa = fma_tab(PT::Ac[i * n + j], in[j], sa);
              }
              om[rr][i] = sm;
              oa[rr][i] = sa;
            }
          }
        }
        __syncthreads();
#pragma unroll
        for (int rr = 0; rr < RA; ++rr) {
          const int task = rr * NT + tid;
          const int q = task / (n * n), r = task - q * (n * n);
          const int j2 = r / n, j1 = r - j2 * n;
          if (task < NA && q < P) {
            if constexpr (L::PR) {
              const int o = lds_base(j1 * SJP2 + (q * n + j2) * m);
#pragma unroll
              for (int i = 0; i < m; ++i) PP[o + i] = T2{om[rr][i], oa[rr][i]};
            } else {
              const int o = lds_base(j1 * SJ1 + (q * n + j2) * m);
#pragma unroll
              for (int i = 0; i < m; ++i) {
                PM[o + i] = om[rr][i];
                PA[o + i] = oa[rr][i];
              }
            }
          }
        }
      } else
      for (int base = 0; base < PPW * n * n; base += NT) {
        const int task = base + tid;
        const int q = task / (n * n), r = task - q * (n * n);
        const int j2 = r / n, j1 = r - j2 * n;
        if (task < PPW * n * n && q < P) {
          T in[n];
          const int row = lds_base((j2 * n + j1) * RS + 2 * K * q);
#pragma unroll
          for (int j = 0; j < n; ++j) in[j] = X[row + j];
          const int o = lds_base(j1 * SJ1 + (q * n + j2) * m);
#pragma unroll
          for (int i = 0; i < m; ++i) {
            T sm = T(0);
#pragma unroll
            for (int j = 0; j < n; ++j) sm = fma_tab(PT::Mc[i * n + j], in[j], sm);
            PM[o + i] = sm;
          }
#pragma unroll
          for (int i = 0; i < m; ++i) {
            T sa = T(0);
#pragma unroll
            for (int j = 0; j < n; ++j) sa = fma_tab(PT::Ac[i * n + j], in[j], sa);
            PA[o + i] = sa;
          }
        }
      }
      __syncthreads();
      // ---- contract x1: lines (q, j2, i0), i0 fastest; U = M1 (M0 x), V = A1 (M0 x) + M1 (A0 x)
      T* U = smem + L::offUV;  // [j2][q][i1][i0]
      T* V = U + n * SJ2;
      if constexpr (L::AL) {
        // aliased: U/V overwrite PM/PA once every line has been read
        constexpr int NB2 = PPW * n * m, RB2 = (NB2 + NT - 1) / NT;
        T ou[RB2][m], ov[RB2][m];
#pragma unroll
        for (int rr = 0; rr < RB2; ++rr) {
          const int task = rr * NT + tid;
          const int q = task / (n * m);
          if (task < NB2 && q < P) {
            T pm[n], pa[n];
#pragma unroll
            for (int j = 0; j < n; ++j) {
              if constexpr (L::PR) {
                const T2 v = PP[j * SJP2 + task];
                pm[j] = v.x;
                pa[j] = v.y;
              } else {
                pm[j] = PM[j * SJ1 + task];
                pa[j] = PA[j * SJ1 + task];
              }
            }
#pragma unroll
            for (int i = 0; i < m; ++i) {
              T su = T(0), sv = T(0);
#pragma unroll
              for (int j = 0; j < n; ++j) {
                su = fma_tab(PT::Mc[i * n + j], pm[j], su);
                sv = fma_tab(PT::Ac[i * n + j], pm[j], sv);
                sv = fma_tab(PT::Mc[i * n + j], pa[j], sv);
              }
              ou[rr][i] = su;
              ov[rr][i] = sv;
            }
          }
        }
        __syncthreads();
#pragma unroll
        for (int rr = 0; rr < RB2; ++rr) {
          const int task = rr * NT + tid;
          const int q = task / (n * m), r = task - q * (n * m);
          const int j2 = r / m, i0 = r - j2 * m;
          if (task < NB2 && q < P) {
            const int o = lds_base(j2 * SJ2 + q * mm + i0);
#pragma unroll
            for (int i = 0; i < m; ++i) {
              U[o + i * m] = ou[rr][i];
              V[o + i * m] = ov[rr][i];
            }
          }
        }
      } else
      for (int base = 0; base < PPW * n * m; base += NT) {
        const int task = base + tid;
        const int q = task / (n * m), r = task - q * (n * m);
        const int j2 = r / m, i0 = r - j2 * m;
        if (task < PPW * n * m && q < P) {
          T pm[n], pa[n];
          const int ri = task;  // = (q * n + j2) * m + i0
#pragma unroll
          for (int j = 0; j < n; ++j) {
            pm[j] = PM[j * SJ1 + ri];
            pa[j] = PA[j * SJ1 + ri];
          }
          const int o = lds_base(j2 * SJ2 + q * mm + i0);
#pragma unroll
          for (int i = 0; i < m; ++i) {
            T su = T(0), sv = T(0);
#pragma unroll
            for (int j = 0; j < n; ++j) {
              su = fma_tab(PT::Mc[i * n + j], pm[j], su);
              sv = fma_tab(PT::Ac[i * n + j], pm[j], sv);
              sv = fma_tab(PT::Mc[i * n + j], pa[j], sv);
            }
            U[o + i * m] = su;
            V[o + i * m] = sv;
          }
        }
      }
      __syncthreads();
    }
    // ---- contract x2 (residual) and apply Sᵀ along x2: lines (q, i1, i0), i0 fastest.  Paired
    // layout: W4 overwrites U/V, so every line is computed before the workgroup synchronises and
    // writes.
    T* W4 = smem + L::offW46;  // [i1][q][a2][i0]
    T tc[RB][m];
#pragma unroll
    for (int rr = 0; rr < RB; ++rr) {
      const int task = rr * NT + tid;
      const int q = task / mm, r = task - q * mm;
      const int i1 = r / m, i0 = r - i1 * m;
      if (task < NB && q < P) {
        T res[m];
        {
          const T* U = smem + L::offUV;
          const T* V = U + n * SJ2;
          T u[n], v[n];
#pragma unroll
          for (int j = 0; j < n; ++j) {
            u[j] = U[j * SJ2 + task];
            v[j] = V[j * SJ2 + task];
          }
#pragma unroll
          for (int i = 0; i < m; ++i) {
            T s = T(0);
#pragma unroll
            for (int j = 0; j < n; ++j) {
              s = fma_tab(PT::Ac[i * n + j], u[j], s);
              s = fma_tab(PT::Mc[i * n + j], v[j], s);
            }
            res[i] = fma(-res_scale, s, bpre[rr][i]);
          }
        }
        apply_st<T, K>(res, tc[rr]);
        if constexpr (!L::PR) {
          const int o = lds_base(i1 * SI1 + q * mm + i0);
#pragma unroll
          for (int a = 0; a < m; ++a) W4[o + a * m] = tc[rr][a];
        }
      }
    }
    if constexpr (L::PR) {
      __syncthreads();
#pragma unroll
      for (int rr = 0; rr < RB; ++rr) {
        const int task = rr * NT + tid;
        const int q = task / mm, r = task - q * mm;
        const int i1 = r / m, i0 = r - i1 * m;
        if (task < NB && q < P) {
          const int o = lds_base(i1 * SI1 + q * mm + i0);
#pragma unroll
          for (int a = 0; a < m; ++a) W4[o + a * m] = tc[rr][a];
        }
      }
    }
    __syncthreads();
    // ---- Sᵀ along x1: lines (q, a2, i0), i0 fastest
    T* W5 = smem + L::offW57;  // [i0][q][a2][a1]
    for (int base = 0; base < PPW * mm; base += NT) {
      const int task = base + tid;
      const int q = task / mm, r = task - q * mm;
      const int a2 = r / m, i0 = r - a2 * m;
      if (task < PPW * mm && q < P) {
        T in[m];
#pragma unroll
        for (int i = 0; i < m; ++i) in[i] = W4[i * SI1 + task];
        const int o = lds_base(i0 * SI0 + q * mm + a2 * m);
        T t[m];
        apply_st<T, K>(in, t);
#pragma unroll
        for (int a = 0; a < m; ++a) W5[o + a] = t[a];
      }
    }
    __syncthreads();
    // ---- Sᵀ along x0, scale by 1/(lam2+lam1+lam0), S along x0: lines (q, a2, a1), a1 fastest
    T* W6 = smem + L::offW46;  // [a1][q][a2][i0]
    for (int base = 0; base < PPW * mm; base += NT) {
      const int task = base + tid;
      const int q = task / mm, r = task - q * mm;
      const int a2 = r / m, a1 = r - a2 * m;
      if (task < PPW * mm && q < P) {
        const DevTables<T>& tb = tab_fresh<T>(K);
        T in[m], z[m];
#pragma unroll
        for (int i = 0; i < m; ++i) in[i] = W5[i * SI0 + task];
        const int li = (a2 * m + a1) * m;
        apply_st<T, K>(in, z);
#pragma unroll
        for (int a = 0; a < m; ++a) z[a] *= tb.inv3[li + a];
        const int o = lds_base(a1 * SA1 + q * mm + a2 * m);
        T w[m];
        apply_s<T, K>(z, w);
#pragma unroll
        for (int i = 0; i < m; ++i) W6[o + i] = w[i];
      }
    }
    __syncthreads();
    // ---- S along x1: lines (q, a2, i0), i0 fastest
    T* W7 = smem + L::offW57;  // [a2][q][i1][i0]
    for (int base = 0; base < PPW * mm; base += NT) {
      const int task = base + tid;
      const int q = task / mm, r = task - q * mm;
      const int a2 = r / m, i0 = r - a2 * m;
      if (task < PPW * mm && q < P) {
        T in[m];
#pragma unroll
        for (int a = 0; a < m; ++a) in[a] = W6[a * SA1 + task];
        const int o = lds_base(a2 * SA2 + q * mm + i0);
        T w[m];
        apply_s<T, K>(in, w);
#pragma unroll
        for (int i = 0; i < m; ++i) W7[o + i * m] = w[i];
      }
    }
    __syncthreads();
    // ---- S along x2 and x^I += correction, straight to global: lines (q, i1, i0)
#pragma unroll
    for (int rr = 0; rr < RB; ++rr) {
      const int task = rr * NT + tid;
      const int q = task / mm;
      if (task < NB && q < P) {
        T in[m];
#pragma unroll
        for (int a = 0; a < m; ++a) in[a] = W7[a * SA2 + task];
        T w[m];
        apply_s<T, K>(in, w);
#pragma unroll
        for (int i = 0; i < m; ++i)
          st_lane(xo + (1 + i) * ld2, loff[rr], fma(sol_scale, w[i], xpre[rr][i]));
      }
    }
  } else {
    // ================================ 2D =====================================
    constexpr int T1 = L::T1, T0 = L::T0, TA = L::TA;
    {
      const T* X = smem + L::offX2;
      T* PM = smem + L::offP2;  // [j1][q][i0]
      T* PA = PM + n * T1;
      // ---- contract x0 with Mc and Ac: lines (q, j1), q fastest
      if constexpr (L::AL2) {
        // aliased: every line is read and contracted, then PM/PA overwrite X
        constexpr int R0 = (PPW * n + NT - 1) / NT;
        T om[R0][m], oa[R0][m];
#pragma unroll
        for (int rr = 0; rr < R0; ++rr) {
          const int task = rr * NT + tid;
          const int j1 = task / PPW, q = task - j1 * PPW;
          if (task < PPW * n && q < P) {
            T in[n];
#pragma unroll
            for (int j = 0; j < n; ++j) in[j] = X[j1 * RS + 2 * K * q + j];
#pragma unroll
            for (int i = 0; i < m; ++i) {
              T sm = T(0), sa = T(0);
#pragma unroll
              for (int j = 0; j < n; ++j) {
                sm = fma_tab(PT::Mc[i * n + j], in[j], sm);
                sa = fma_tab(PT::Ac[i * n + j], in[j], sa);
              }
              om[rr][i] = sm;
              oa[rr][i] = sa;
            }
          }
        }
        __syncthreads();
#pragma unroll
        for (int rr = 0; rr < R0; ++rr) {
          const int task = rr * NT + tid;
          const int j1 = task / PPW, q = task - j1 * PPW;
          if (task < PPW * n && q < P) {
            const int o = lds_base(j1 * T1 + q * m);
#pragma unroll
            for (int i = 0; i < m; ++i) {
              PM[o + i] = om[rr][i];
              PA[o + i] = oa[rr][i];
            }
          }
        }
      } else
      for (int base = 0; base < PPW * n; base += NT) {
        const int task = base + tid;
        const int j1 = task / PPW, q = task - j1 * PPW;
        if (task < PPW * n && q < P) {
          T in[n];
#pragma unroll
          for (int j = 0; j < n; ++j) in[j] = X[j1 * RS + 2 * K * q + j];
          const int o = lds_base(j1 * T1 + q * m);
#pragma unroll
          for (int i = 0; i < m; ++i) {
            T sm = T(0);
#pragma unroll
            for (int j = 0; j < n; ++j) sm = fma_tab(PT::Mc[i * n + j], in[j], sm);
            PM[o + i] = sm;
          }
#pragma unroll
          for (int i = 0; i < m; ++i) {
            T sa = T(0);
#pragma unroll
            for (int j = 0; j < n; ++j) sa = fma_tab(PT::Ac[i * n + j], in[j], sa);
            PA[o + i] = sa;
          }
        }
      }
      __syncthreads();
    }
    // ---- residual along x1, r = b - (A1 (M0 x) + M1 (A0 x)) , then Sᵀ along x1:
    //      lines (q, i0), i0 fastest.  Aliased layout: W overwrites PM/PA, so every line is
    //      computed before the workgroup synchronises and writes.
    T* W = smem + L::offW;  // [i0][q][a1]
    T tw[RB][m];
#pragma unroll
    for (int rr = 0; rr < RB; ++rr) {
      const int task = rr * NT + tid;
      const int q = task / m;
      if (task < NB && q < P) {
        T res[m];
        {
          const T* PM = smem + L::offP2;
          const T* PA = PM + n * T1;
          T pm[n], pa[n];
#pragma unroll
          for (int j = 0; j < n; ++j) {
            pm[j] = PM[j * T1 + task];
            pa[j] = PA[j * T1 + task];
          }
#pragma unroll
          for (int i = 0; i < m; ++i) {
            T s = T(0);
#pragma unroll
            for (int j = 0; j < n; ++j) {
              s = fma_tab(PT::Ac[i * n + j], pm[j], s);
              s = fma_tab(PT::Mc[i * n + j], pa[j], s);
            }
            res[i] = fma(-res_scale, s, bpre[rr][i]);
          }
        }
        apply_st<T, K>(res, tw[rr]);
      }
    }
    if constexpr (L::AL2) __syncthreads();
#pragma unroll
    for (int rr = 0; rr < RB; ++rr) {
      const int task = rr * NT + tid;
      const int q = task / m, i0 = task - q * m;
      if (task < NB && q < P) {
        const int o = lds_base(i0 * T0 + q * m);
#pragma unroll
        for (int a = 0; a < m; ++a) W[o + a] = tw[rr][a];
      }
    }
    __syncthreads();
    // ---- Sᵀ along x0, scale by 1/(lam1+lam0), S along x0: lines (q, a1), a1 fastest
    T* W2 = smem + L::offW2;  // [a1][q][i0]
    for (int base = 0; base < PPW * m; base += NT) {
      const int task = base + tid;
      const int q = task / m, a1 = task - q * m;
      if (task < PPW * m && q < P) {
        const DevTables<T>& tb = tab_fresh<T>(K);
        T in[m], z[m];
#pragma unroll
        for (int i = 0; i < m; ++i) in[i] = W[i * T0 + task];
        apply_st<T, K>(in, z);
#pragma unroll
        for (int a = 0; a < m; ++a) z[a] *= tb.inv2[a1 * m + a];
        const int o = lds_base(a1 * TA + q * m);
        T w[m];
        apply_s<T, K>(z, w);
#pragma unroll
        for (int i = 0; i < m; ++i) W2[o + i] = w[i];
      }
    }
    __syncthreads();
    // ---- S along x1 and x^I += correction, straight to global: lines (q, i0)
#pragma unroll
    for (int rr = 0; rr < RB; ++rr) {
      const int task = rr * NT + tid;
      const int q = task / m;
      if (task < NB && q < P) {
        T in[m];
#pragma unroll
        for (int a = 0; a < m; ++a) in[a] = W2[a * TA + task];
        T w[m];
        apply_s<T, K>(in, w);
#pragma unroll
        for (int i = 0; i < m; ++i)
          st_lane(xo + (1 + i) * ld1, loff[rr], fma(sol_scale, w[i], xpre[rr][i]));
      }
    }
  }
}

// ------------------------------------------------------------------ matrix-core form (3D, FP32)
//
// The three contractions of the localised residual r = b - Abar x (Sec. 3.1.1) are dense products
// of a batch of patch lines with one small 1D matrix, so they run on the matrix cores
// (v_mfma_f32_16x16x4f32: 16 lines x 4 inputs times 4 inputs x 16 outputs, FP32 products
// accumulated in FP32); the fast-diagonalisation stages stay on the vector ALU, where the
// eigenvectors' mirror symmetry halves their multiply-adds.  Lines of the workgroup's PPW
// patches are stacked into 16-row tiles; the 1D matrices sit in per-lane registers (B operand):
//   x0: lines (q, j2, j1) of the closure, inputs c (n, padded to a multiple of 4), outputs
//       [M0 x | A0 x] (2m <= 16)                                  -> PM, PA [i0][line]
//   x1: lines (q, i0, j2), inputs [PM(j1) | PA(j1)] (2n), outputs
//       [M1 PM | A1 PM + M1 PA] (2m)                               -> U, V  [i1][line]
//   x2: lines (q, i1, i0), inputs [U(j2) | V(j2)] (2n), outputs A2 U + M2 V (m); the vector ALU
//       then forms r = b - h (A2 U + M2 V) and applies S^T along x2, as in colour_pass_lines.
// Matrix-core operand layout (16x16x4, FP32): lane l holds A[l % 16][l / 16] and B[l / 16][l % 16]
// and receives D[4 (l / 16) + i][l % 16] in accumulator register i.
template <int K, int PPW>
struct MfmaLds {
  static constexpr int n = 2 * K + 1, m = 2 * K - 1, mm = m * m, nn = n * n;
  static constexpr int KB0 = (n + 3) / 4, KB1 = (2 * n + 3) / 4;     // 4-wide input blocks
  static constexpr int R0 = PPW * nn, R1 = PPW * m * n, R2 = PPW * mm;  // lines per stage
  static constexpr int T0 = (R0 + 15) / 16, T1 = (R1 + 15) / 16, T2 = (R2 + 15) / 16;
  static constexpr int RS = 2 * K * PPW + 1;
  // closure rows padded so that a tile's 4-wide input blocks past column n stay inside the row (their
  // B rows are zero; the values read there are zeros written by the closure load), and = 4 (mod 32)
  // so that the 16 rows of a tile fall into distinct bank groups
  static constexpr int RSX = pad32(RS + 4 * KB0 - n, 4);
  static constexpr int LS0 = pad32(16 * T0, 20);   // PM / PA row: tile writes of 4 lines at once
  static constexpr int LS1 = pad32(16 * T1, 4);    // U / V row
  static constexpr int LS2 = pad32(16 * T2, 4);    // x2 result row
  static constexpr int X = nn * RSX;
  static constexpr int P = 2 * m * LS0;            // PM, PA
  static constexpr int UV = 2 * m * LS1;           // U, V
  static constexpr int Q = m * LS2;                // A2 U + M2 V
  using Fd = SmootherLds<3, K, float, PPW>;  // strides of the diagonalisation stages
  static constexpr int FD = m * (Fd::SI1 > Fd::SI0 ? (Fd::SI1 > Fd::SA1 ? (Fd::SI1 > Fd::SA2 ? Fd::SI1 : Fd::SA2)
                                                                         : (Fd::SA1 > Fd::SA2 ? Fd::SA1 : Fd::SA2))
                                                   : (Fd::SI0 > Fd::SA1 ? (Fd::SI0 > Fd::SA2 ? Fd::SI0 : Fd::SA2)
                                                                         : (Fd::SA1 > Fd::SA2 ? Fd::SA1 : Fd::SA2)));
  static constexpr int max2(int a, int b) { return a > b ? a : b; }
  // region 0: X, then U/V, then the diagonalisation buffers of odd stages; region 1: PM/PA, then Q,
  // then the even ones
  static constexpr int A = max2(max2(X, UV), FD);
  static constexpr int B = max2(max2(P, Q), FD);
  static constexpr int total = A + B;
};

typedef float vps_f32x4 __attribute__((ext_vector_type(4)));

template <int K, int PPW>
__device__ __forceinline__ void colour_pass_mfma3(float* __restrict__ smem, const float* __restrict__ b,
                                                  float* __restrict__ x, long long n1d, int p0, int p1, int p2,
                                                  int cnt0, int cnt1, int groups0, float res_scale, float sol_scale,
                                                  unsigned blk) {
  using L = MfmaLds<K, PPW>;
  using PT = gen::PatchTables<float, K>;
  using Fd = typename L::Fd;
  constexpr int n = L::n, m = L::m, mm = L::mm, nn = L::nn, RS = L::RS, RSX = L::RSX;
  constexpr int NT = 256, NW = NT / 64;
  static_assert(2 * m <= 16, "outputs of one contraction must fit the 16 matrix columns");
  float* const rA = smem;         // X, then U/V, then odd diagonalisation buffers
  float* const rB = smem + L::A;  // PM/PA, then Q, then even ones

  const ColourBlock cb = colour_block<3, K, PPW>(blk, p0, p1, p2, cnt0, cnt1, groups0);
  const int P = cb.count;
  const long long s0 = cb.s0, s1 = cb.s1, s2 = cb.s2;
  const long long n1d2 = n1d * n1d;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 15, lk = lane >> 4;  // matrix-core row (A) / column (B, D) and input sub-index
  const int seg = 2 * K * P + 1;             // valid closure columns along x0
  const int ld1 = (int)n1d, ld2 = (int)n1d2;
  float* xo = x + (s2 * n1d2 + s1 * n1d + s0);
  const float* bo = b + (s2 * n1d2 + s1 * n1d + s0);

  // B operands (1D patch matrices; zero rows pad the inputs, zero columns the outputs)
  float bx0[L::KB0], bx1[L::KB1], bx2[L::KB1];
#pragma unroll
  for (int kb = 0; kb < L::KB0; ++kb) {
    const int k = 4 * kb + lk;
    bx0[kb] = k >= n ? 0.f : lr < m ? PT::Mc[lr * n + k] : lr < 2 * m ? PT::Ac[(lr - m) * n + k] : 0.f;
  }
#pragma unroll
  for (int kb = 0; kb < L::KB1; ++kb) {
    const int k = 4 * kb + lk;
    const bool pm = k < n, pa = k >= n && k < 2 * n;
    const int c = pm ? k : k - n;
    bx1[kb] = lr < m ? (pm ? PT::Mc[lr * n + c] : 0.f)
                     : lr < 2 * m ? (pm ? PT::Ac[(lr - m) * n + c] : pa ? PT::Mc[(lr - m) * n + c] : 0.f) : 0.f;
    bx2[kb] = lr < m ? (pm ? PT::Ac[lr * n + c] : pa ? PT::Mc[lr * n + c] : 0.f) : 0.f;
  }

  // Lines (q, i1, i0) of the vector stages: b on them is prefetched now (tasks past the last patch
  // are clamped to it, so every load is in bounds)
  constexpr int NB = PPW * mm;
  constexpr int RB = (NB + NT - 1) / NT;
  float bpre[RB][m], xpre[RB][m];
  unsigned loff[RB];
  int xoff[RB];
#pragma unroll
  for (int rr = 0; rr < RB; ++rr) {
    const int task = rr * NT + tid;
    int q = task / mm;
    const int r = task - q * mm, i1 = r / m, i0 = r - i1 * m;
    q = min(q, P - 1);
    loff[rr] = (unsigned)((1 + i1) * ld1 + 2 * K * q + 1 + i0) * (unsigned)sizeof(float);
    xoff[rr] = (n + 1 + i1) * RSX + 2 * K * q + 1 + i0;  // node (i = 0) in the LDS closure
#pragma unroll
    for (int i = 0; i < m; ++i) bpre[rr][i] = ld_lane(bo + ld2 + i * ld2, loff[rr]);
  }

  // ---- closure -> X [j2][j1][c]; Dirichlet nodes, and columns past the workgroup's last patch, are 0
  {
    float* X = rA;
    const bool lo1 = s1 == 0, hi1 = s1 + n - 1 == n1d - 1;
    const bool lo2 = s2 == 0, hi2 = s2 + n - 1 == n1d - 1;
    for (int w = tid; w < RSX * n; w += NT) {
      const int j1 = w / RSX, c = w - j1 * RSX;
      const int cl = min(c, seg - 1);
      const long long gc = s0 + cl;
      const bool bad = c >= seg || gc == 0 || gc == n1d - 1 || (j1 == 0 && lo1) || (j1 == n - 1 && hi1);
      const unsigned base = (unsigned)(j1 * ld1 + cl) * (unsigned)sizeof(float);
      float v[n];
#pragma unroll
      for (int j = 0; j < n; ++j) v[j] = ld_lane(xo + j * ld2, base);
#pragma unroll
      for (int j = 0; j < n; ++j) {
        const bool zero = bad || (j == 0 && lo2) || (j == n - 1 && hi2);
        X[(j * n + j1) * RSX + c] = zero ? 0.f : v[j];
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int rr = 0; rr < RB; ++rr) {
#pragma unroll
    for (int i = 0; i < m; ++i) xpre[rr][i] = rA[xoff[rr] + i * n * RSX];  // old x^I (never Dirichlet)
  }

  // ---- x0 on the matrix cores: lines (q, j2, j1) -> PM, PA [i0][line]
  {
    const float* X = rA;
    float* PM = rB;
    for (int t = wave; t < L::T0; t += NW) {
      const int row = min(16 * t + lr, L::R0 - 1);
      const int q = row / nn, rem = row - q * nn;
      const int a = lds_base(rem * RSX + 2 * K * q + lk);
      vps_f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kb = 0; kb < L::KB0; ++kb) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(X[a + 4 * kb], bx0[kb], acc, 0, 0, 0);
      if (lr < 2 * m) *reinterpret_cast<vps_f32x4*>(PM + lr * L::LS0 + 16 * t + 4 * lk) = acc;
    }
  }
  __syncthreads();
  // ---- x1 on the matrix cores: lines (q, i0, j2), inputs PM(j1), PA(j1) -> U, V [i1][line]
  {
    const float* PM = rB;
    float* U = rA;
    int koff[L::KB1];
#pragma unroll
    for (int kb = 0; kb < L::KB1; ++kb) {
      const int k = 4 * kb + lk;
      koff[kb] = k < n ? k : k < 2 * n ? m * L::LS0 + (k - n) : 0;
    }
    for (int t = wave; t < L::T1; t += NW) {
      const int row = min(16 * t + lr, L::R1 - 1);
      const int q = row / (m * n), rem = row - q * (m * n);
      const int i0 = rem / n, j2 = rem - i0 * n;
      const int a = lds_base(i0 * L::LS0 + q * nn + j2 * n);
      vps_f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kb = 0; kb < L::KB1; ++kb) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(PM[a + koff[kb]], bx1[kb], acc, 0, 0, 0);
      if (lr < 2 * m) *reinterpret_cast<vps_f32x4*>(U + lr * L::LS1 + 16 * t + 4 * lk) = acc;
    }
  }
  __syncthreads();
  // ---- x2 on the matrix cores: lines (q, i1, i0), inputs U(j2), V(j2) -> Q = A2 U + M2 V [i2][line]
  {
    const float* U = rA;
    float* Q = rB;
    int koff[L::KB1];
#pragma unroll
    for (int kb = 0; kb < L::KB1; ++kb) {
      const int k = 4 * kb + lk;
      koff[kb] = k < n ? k : k < 2 * n ? m * L::LS1 + (k - n) : 0;
    }
    for (int t = wave; t < L::T2; t += NW) {
      const int row = min(16 * t + lr, L::R2 - 1);
      const int q = row / mm, rem = row - q * mm;
      const int i1 = rem / m, i0 = rem - i1 * m;
      const int a = lds_base(i1 * L::LS1 + (q * m + i0) * n);
      vps_f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kb = 0; kb < L::KB1; ++kb) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(U[a + koff[kb]], bx2[kb], acc, 0, 0, 0);
      if (lr < m) *reinterpret_cast<vps_f32x4*>(Q + lr * L::LS2 + 16 * t + 4 * lk) = acc;
    }
  }
  __syncthreads();

  constexpr int SI1 = Fd::SI1, SI0 = Fd::SI0, SA1 = Fd::SA1, SA2 = Fd::SA2;
  // ---- r = b - h (A2 U + M2 V), then S^T along x2: lines (q, i1, i0)
  {
    const float* Q = rB;
    float* W4 = rA;  // [i1][q][a2][i0]
#pragma unroll
    for (int rr = 0; rr < RB; ++rr) {
      const int task = rr * NT + tid;
      const int q = task / mm, r = task - q * mm;
      const int i1 = r / m, i0 = r - i1 * m;
      if (task < NB && q < P) {
        float res[m];
#pragma unroll
        for (int i = 0; i < m; ++i) res[i] = fma(-res_scale, Q[i * L::LS2 + task], bpre[rr][i]);
        float t[m];
        apply_st<float, K>(res, t);
        const int o = lds_base(i1 * SI1 + q * mm + i0);
#pragma unroll
        for (int a = 0; a < m; ++a) W4[o + a * m] = t[a];
      }
    }
  }
  __syncthreads();
  // ---- S^T along x1: lines (q, a2, i0)
  {
    const float* W4 = rA;
    float* W5 = rB;  // [i0][q][a2][a1]
    for (int base = 0; base < PPW * mm; base += NT) {
      const int task = base + tid;
      const int q = task / mm, r = task - q * mm;
      const int a2 = r / m, i0 = r - a2 * m;
      if (task < PPW * mm && q < P) {
        float in[m];
#pragma unroll
        for (int i = 0; i < m; ++i) in[i] = W4[i * SI1 + task];
        const int o = lds_base(i0 * SI0 + q * mm + a2 * m);
        float t[m];
        apply_st<float, K>(in, t);
#pragma unroll
        for (int a = 0; a < m; ++a) W5[o + a] = t[a];
      }
    }
  }
  __syncthreads();
  // ---- S^T along x0, 1/(lam2 + lam1 + lam0), S along x0: lines (q, a2, a1)
  {
    const float* W5 = rB;
    float* W6 = rA;  // [a1][q][a2][i0]
    for (int base = 0; base < PPW * mm; base += NT) {
      const int task = base + tid;
      const int q = task / mm, r = task - q * mm;
      const int a2 = r / m, a1 = r - a2 * m;
      if (task < PPW * mm && q < P) {
        const DevTables<float>& tb = tab_fresh<float>(K);
        float in[m], z[m];
#pragma unroll
        for (int i = 0; i < m; ++i) in[i] = W5[i * SI0 + task];
        const int li = (a2 * m + a1) * m;
        apply_st<float, K>(in, z);
#pragma unroll
        for (int a = 0; a < m; ++a) z[a] *= tb.inv3[li + a];
        const int o = lds_base(a1 * SA1 + q * mm + a2 * m);
        float w[m];
        apply_s<float, K>(z, w);
#pragma unroll
        for (int i = 0; i < m; ++i) W6[o + i] = w[i];
      }
    }
  }
  __syncthreads();
  // ---- S along x1: lines (q, a2, i0)
  {
    const float* W6 = rA;
    float* W7 = rB;  // [a2][q][i1][i0]
    for (int base = 0; base < PPW * mm; base += NT) {
      const int task = base + tid;
      const int q = task / mm, r = task - q * mm;
      const int a2 = r / m, i0 = r - a2 * m;
      if (task < PPW * mm && q < P) {
        float in[m];
#pragma unroll
        for (int a = 0; a < m; ++a) in[a] = W6[a * SA1 + task];
        const int o = lds_base(a2 * SA2 + q * mm + i0);
        float w[m];
        apply_s<float, K>(in, w);
#pragma unroll
        for (int i = 0; i < m; ++i) W7[o + i * m] = w[i];
      }
    }
  }
  __syncthreads();
  // ---- S along x2 and x^I += correction / h, straight to global: lines (q, i1, i0)
  {
    const float* W7 = rB;
#pragma unroll
    for (int rr = 0; rr < RB; ++rr) {
      const int task = rr * NT + tid;
      const int q = task / mm;
      if (task < NB && q < P) {
        float in[m];
#pragma unroll
        for (int a = 0; a < m; ++a) in[a] = W7[a * SA2 + task];
        float w[m];
        apply_s<float, K>(in, w);
#pragma unroll
        for (int i = 0; i < m; ++i) st_lane(xo + (1 + i) * ld2, loff[rr], fma(sol_scale, w[i], xpre[rr][i]));
      }
    }
  }
}

// Patches per workgroup of the matrix-core form (3D Q4, FP32, multiplicative), 256 threads.
constexpr int kMfmaPPW = 4;
template <int D, int K, typename T>
struct HasMfmaForm {
  static constexpr bool value = D == 3 && K == 4 && sizeof(T) == 4;
};

// What one workgroup of a launch runs, per mode and shape: SH is an EigShape for the eigenbasis form
// (multiplicative and Boundary), else a LineShape.
template <int PPWv, int NTv>
struct LineShape {
  static constexpr int PPW = PPWv, NT = NTv;
};
template <int D, int K, typename T, int MODE, typename SH>
struct ColourBody {
  // the residual form of the 3D pass in FP64 contracts the closure along x2 first, where it measured 3-9%
  // faster than the closure-through-LDS form; in FP32 the two measured within 2%
  static_assert(MODE == kModeResidual, "line shapes serve the residual form");
  static constexpr bool kMult3 = D == 3 && sizeof(T) == 8;
  static constexpr int lds() {
    if constexpr (kMult3) return Mult3Lds<K, SH::PPW>::total;
    else return SmootherLds<D, K, T, SH::PPW, LinesAlias<D, K, T, MODE, SH::PPW>::value,
                            LinesPair<D, K, T, MODE, SH::PPW>::value>::total;
  }
  static constexpr int kLds = lds();
  static __device__ __forceinline__ void run(T* smem, const T* b, T* x, long long n1d, int p0, int p1, int p2, int cnt0,
                                             int cnt1, int groups0, T res_scale, T sol_scale, unsigned blk) {
    if constexpr (kMult3)
      colour_pass_mult3<K, T, SH::PPW>(smem, b, x, n1d, p0, p1, p2, cnt0, cnt1, groups0, res_scale, sol_scale, blk);
    else
      colour_pass_lines<D, K, T, MODE, SH::PPW>(smem, b, x, n1d, p0, p1, p2, cnt0, cnt1, groups0, res_scale, sol_scale,
                                                blk);
  }
};
template <int D, int K, typename T, int MODE, int PPW, int NT, bool AL>
struct ColourBody<D, K, T, MODE, EigShape<PPW, NT, AL>> {
  using SH = EigShape<PPW, NT, AL>;
  static constexpr bool kPoison = MODE == kModeMultiplicative;
  static constexpr int lds() {
    if constexpr (D == 3) return EigLds3<K, SH>::total;
    else return EigLds2<K, SH>::total;
  }
  static constexpr int kLds = lds();
  static __device__ __forceinline__ void run_team(T* smem, int tid, bool active, const T* b, T* x, long long n1d, int p0,
                                                  int p1, int p2, int cnt0, int cnt1, int groups0, T, T sol_scale,
                                                  unsigned blk) {
    if constexpr (D == 3)
      colour_pass_eig3<K, T, kPoison, SH>(smem, b, x, n1d, p0, p1, p2, cnt0, cnt1, groups0, sol_scale, blk, tid, active);
    else
      colour_pass_eig2<K, T, kPoison, SH>(smem, b, x, n1d, p0, p1, cnt0, cnt1, groups0, sol_scale, blk, tid, active);
  }
  static __device__ __forceinline__ void run(T* smem, const T* b, T* x, long long n1d, int p0, int p1, int p2, int cnt0,
                                             int cnt1, int groups0, T res_scale, T sol_scale, unsigned blk) {
    run_team(smem, threadIdx.x, true, b, x, n1d, p0, p1, p2, cnt0, cnt1, groups0, res_scale, sol_scale, blk);
  }
};
template <int D, int K, typename T, bool ZERO, typename SH>
struct AddBody {
  static constexpr int kLds = AddLds<D, K, SH>::total;
  static __device__ __forceinline__ void run_team(T* smem, int tid, bool active, const T* b, T* x, long long n1d, int p0,
                                                  int p1, int p2, int cnt0, int cnt1, int groups0, T, T sol_scale,
                                                  unsigned blk) {
    colour_pass_add<D, K, T, ZERO, SH>(smem, b, x, n1d, p0, p1, p2, cnt0, cnt1, groups0, sol_scale, blk, tid, active);
  }
  static __device__ __forceinline__ void run(T* smem, const T* b, T* x, long long n1d, int p0, int p1, int p2, int cnt0,
                                             int cnt1, int groups0, T res_scale, T sol_scale, unsigned blk) {
    run_team(smem, threadIdx.x, true, b, x, n1d, p0, p1, p2, cnt0, cnt1, groups0, res_scale, sol_scale, blk);
  }
};
template <int D, int K, typename T, int PPW, int NT, bool AL>
struct ColourBody<D, K, T, kModeAdditive, EigShape<PPW, NT, AL>> : AddBody<D, K, T, false, EigShape<PPW, NT, AL>> {};
template <int D, int K, typename T, int PPW, int NT, bool AL>
struct ColourBody<D, K, T, kModeZero, EigShape<PPW, NT, AL>> : AddBody<D, K, T, true, EigShape<PPW, NT, AL>> {};
template <int D, typename T, int MODE, int PPW>
struct ColourBody<D, 1, T, MODE, Q1Shape<PPW>> {
  static constexpr int kLds = 1;
  static __device__ __forceinline__ void run_team(T*, int tid, bool active, const T* b, T* x, long long n1d, int p0, int p1,
                                                  int p2, int cnt0, int cnt1, int groups0, T res_scale, T sol_scale,
                                                  unsigned blk) {
    colour_pass_q1<D, T, MODE == kModeMultiplicative, PPW>(b, x, n1d, p0, p1, p2, cnt0, cnt1, groups0, res_scale,
                                                           sol_scale, blk, tid, active);
  }
  static __device__ __forceinline__ void run(T* smem, const T* b, T* x, long long n1d, int p0, int p1, int p2, int cnt0,
                                             int cnt1, int groups0, T res_scale, T sol_scale, unsigned blk) {
    run_team(smem, threadIdx.x, true, b, x, n1d, p0, p1, p2, cnt0, cnt1, groups0, res_scale, sol_scale, blk);
  }
};
template <int D, int K, int PPW, int NT>
struct ColourBody<D, K, float, kModeMfma, LineShape<PPW, NT>> {
  static constexpr int kLds = MfmaLds<K, PPW>::total;
  static __device__ __forceinline__ void run(float* smem, const float* b, float* x, long long n1d, int p0, int p1, int p2,
                                             int cnt0, int cnt1, int groups0, float res_scale, float sol_scale,
                                             unsigned blk) {
    colour_pass_mfma3<K, PPW>(smem, b, x, n1d, p0, p1, p2, cnt0, cnt1, groups0, res_scale, sol_scale, blk);
  }
};

template <int D, int K, typename T, int MODE, typename SH>
__global__ __launch_bounds__((SH::NT)) void colour_pass_kernel(const T* __restrict__ b, T* __restrict__ x,
                                                               long long n1d, int p0, int p1, int p2, int cnt0,
                                                               int cnt1, int groups0, T res_scale, T sol_scale) {
  using Body = ColourBody<D, K, T, MODE, SH>;
  __shared__ __align__(16) T smem[Body::kLds];
  Body::run(smem, b, x, n1d, p0, p1, p2, cnt0, cnt1, groups0, res_scale, sol_scale,
            xcd_remap(blockIdx.x, gridDim.x));
}

// Several colour passes of the same (dim, degree, precision, colour) on different vectors and
// levels in one launch: entry e owns blocks [begin[e], begin[e+1]).
template <int D, int K, typename T, int MODE, typename SH>
__global__ __launch_bounds__((SH::NT)) void colour_pass_group_kernel(ColourPassGroup grp) {
  using Body = ColourBody<D, K, T, MODE, SH>;
  __shared__ __align__(16) T smem[Body::kLds];
  const unsigned g = xcd_remap(blockIdx.x, gridDim.x);
  int e = 0;
  while (e + 1 < grp.n && (unsigned)grp.e[e + 1].block_begin <= g) ++e;
  const ColourPassDesc& d = grp.e[e];
  Body::run(smem, (const T*)d.b, (T*)d.x, d.n1d, d.p[0], d.p[1], d.p[2], d.cnt0, d.cnt1, d.groups0, (T)d.res_scale,
            (T)d.sol_scale, g - (unsigned)d.block_begin);
}

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

template <int D, int K, typename T, bool ADD>
__global__ __launch_bounds__((FusedTeams<D, K, T>::SH::NT * FusedTeams<D, K, T>::N)) void colour_span_kernel(
    FusedMembers mem, long long n1d, int half, int span, int first, int n_colours, int step, int clear, T res_scale,
    T sol_scale) {
  using SH = typename FusedTeams<D, K, T>::SH;
  using Body = std::conditional_t<ADD, AddBody<D, K, T, false, SH>,
                                  ColourBody<D, K, T, K == 1 ? kModeMultiplicative : kModeBoundary, SH>>;
  constexpr int TEAMS = FusedTeams<D, K, T>::N, NT = SH::NT, PPW = SH::PPW;
  constexpr int kLds = (Body::kLds + 3) & ~3;
  __shared__ __align__(16) T smem[kLds * TEAMS];
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
      Body::run_team(smem + team * kLds, tid, k < per, b, x, n1d, p0, p1, p2, cnt0, cnt1, groups0, res_scale,
                     sol_scale, (unsigned)(w * per + (k < per ? k : 0)));
      __syncthreads();
    }
  }
}

// The exact solve on the coarsest level: one patch, FP64 arithmetic for both precisions, one workgroup per
// member; the boundary nodes of x become 0.  Lines as in the passes above: S^T along x2, x1 and x0, the
// eigenvalue scaling, S along x0, x1 and x2 (2D: x1, x0, x0, x1).
template <int D, int K>
struct CoarseLds {
  static constexpr int m = 2 * K - 1, words = D == 3 ? m * m * m : m * m;  // doubles of one buffer
};
template <int D, int K, typename T, int NT>
__device__ __forceinline__ void coarse_solve(double* __restrict__ w0, double* __restrict__ w1, const T* __restrict__ b,
                                             T* __restrict__ x, int t) {
  constexpr int n = 2 * K + 1, m = 2 * K - 1, mm = m * m, L = D == 3 ? mm : m;
  static_assert(NT >= L, "a line per thread");
  const DevTables<double>& tb = tab<double>(K);
  for (int i = t; i < (D == 3 ? n * n * n : n * n); i += NT) {
    const int i0 = i % n, i1 = (i / n) % n, i2 = i / (n * n);
    if (i0 == 0 || i0 == n - 1 || i1 == 0 || i1 == n - 1 || (D == 3 && (i2 == 0 || i2 == n - 1))) x[i] = T(0);
  }
  // line t of the slowest axis: node (1 + i, 1 + t / m, 1 + t % m) in 3D, (1 + i, 1 + t) in 2D
  const int base = D == 3 ? (1 + t / m) * n + 1 + t % m : 1 + t, st = D == 3 ? n * n : n;
  double v[m], u[m];
  if (t < L) {
#pragma unroll
    for (int i = 0; i < m; ++i) v[i] = (double)b[(1 + i) * st + base];
    apply_st<double, K>(v, u);
#pragma unroll
    for (int a = 0; a < m; ++a) w0[a * L + t] = u[a];
  }
  __syncthreads();
  if constexpr (D == 3) {
    if (t < L) {
      const int a2 = t / m, i0 = t % m;
#pragma unroll
      for (int i = 0; i < m; ++i) v[i] = w0[a2 * L + i * m + i0];
      apply_st<double, K>(v, u);
#pragma unroll
      for (int a = 0; a < m; ++a) w1[a2 * L + a * m + i0] = u[a];
    }
    __syncthreads();
  }
  if (t < L) {
    const double* in = D == 3 ? w1 : w0;  // lines (a2, a1) / a1 along x0
    double* out = D == 3 ? w0 : w1;
#pragma unroll
    for (int i = 0; i < m; ++i) v[i] = in[t * m + i];
    apply_st<double, K>(v, u);
#pragma unroll
    for (int a = 0; a < m; ++a) u[a] *= D == 3 ? tb.inv3[t * m + a] : tb.inv2[t * m + a];
    apply_s<double, K>(u, v);
#pragma unroll
    for (int i = 0; i < m; ++i) out[t * m + i] = v[i];
  }
  __syncthreads();
  if constexpr (D == 3) {
    if (t < L) {
      const int a2 = t / m, i0 = t % m;
#pragma unroll
      for (int a = 0; a < m; ++a) v[a] = w0[a2 * L + a * m + i0];
      apply_s<double, K>(v, u);
#pragma unroll
      for (int i = 0; i < m; ++i) w1[a2 * L + i * m + i0] = u[i];
    }
    __syncthreads();
  }
  if (t < L) {
    constexpr double scale = D == 3 ? 2.0 : 1.0;  // h^(2-d), h = 1/2
#pragma unroll
    for (int a = 0; a < m; ++a) v[a] = w1[a * L + t];
    apply_s<double, K>(v, u);
#pragma unroll
    for (int i = 0; i < m; ++i) x[(1 + i) * st + base] = (T)(scale * u[i]);
  }
}

template <int D, int K, typename T>
__global__ __launch_bounds__(256) void coarse_solve_kernel(FusedMembers mem) {
  __shared__ double w[2 * CoarseLds<D, K>::words];
  coarse_solve<D, K, T, 256>(w, w + CoarseLds<D, K>::words, (const T*)mem.b[blockIdx.x], (T*)mem.x[blockIdx.x],
                             threadIdx.x);
}

// ------------------------------------------------------------------ the small levels of a V-cycle in one launch
//
// The V-cycle from x = 0 on a level of a few thousand nodes is a chain of short stages: as launches each costs
// 2-4 us of which well under 1 us is work.  Here one workgroup per member holds right-hand side, iterate and
// scratch of the levels 1..top in LDS and runs the whole chain, level by level, with barriers only.  A stage then
// costs an LDS round trip, and the launches, the global round trips between the stages and the stores' drain at
// each launch's end go.
// Smoothing: the colour passes of a span of the whole grid, on LdsWindow.  Transfer: with x in the fine space and
// R = P^T, the next right-hand side R b - R A x is summed axis by axis, each axis restricted as it is contracted
// (RA, RM: P^T times the 1D matrices of a coarse cell's two fine cells), so the second and third axis work on half
// and a quarter of the lines.  Measured, device time: 2D degree 3 FP64 level 3 and
// below 38 us against 11 launches of 3.5-8 us and their gaps; 3D degree 2 FP32 level 2 36 us against 7 launches.  What
// bounds it is one workgroup's chain of barriers, LDS round trips and dependent multiply-adds (16 passes of 1.7 us in
// the first case); a copy of the reciprocal tables in LDS changed nothing.  Structure: P's columns of coarse nodes off the boundary vanish on fine boundary
// nodes, so the fine residual's boundary entries never enter; values on coarse boundary nodes are left undefined
// and never read.
template <int D, int K, typename T, int TOP>
struct CycleLds {
  using SH = typename FusedTeams<D, K, T>::SH;
  // four teams cover a colour of level 3 in 2D; with 512 threads a lane has 256 registers
  static constexpr int TEAMS = D == 2 && K >= 4 ? 4 : FusedTeams<D, K, T>::N, NT = TEAMS * SH::NT;
  static constexpr __host__ __device__ int n1d(int l) { return (K << l) + 1; }
  static constexpr __host__ __device__ int stride(int l) {  // words of a level's vector
    return even_up(n1d(l) * n1d(l) * (D == 3 ? n1d(l) : 1));
  }
  static constexpr __host__ __device__ int offset(int l) {  // level l: its iterate, then its right-hand side
    int o = 0;
    for (int i = 1; i < l; ++i) o += 2 * stride(i);
    return o;
  }
  static constexpr int lds_team() {
    if constexpr (K == 1) return 0;
    else if constexpr (D == 3) return (EigLds3<K, SH>::total + 3) & ~3;
    else return (EigLds2<K, SH>::total + 3) & ~3;
  }
  static constexpr int kTeam = lds_team();
  static constexpr int nf = n1d(TOP), nc = n1d(TOP - 1);
  static constexpr int kTransfer = D == 3 ? 3 * nc * nf * (nf + nc) : 3 * nc * nf;
  static constexpr int kCoarse = 2 * CoarseLds<D, K>::words * (int)(8 / sizeof(T));
  static constexpr int work = (offset(TOP + 1) + 3) & ~3;
  static constexpr int total = work + max_of(max_of(kTeam * TEAMS, kTransfer), kCoarse);
  static_assert(total * sizeof(T) <= 160 * 1024, "LDS of a compute unit");
};

// y: coarse nodes K C .. K C + K - 1 of one axis from the fine nodes 2K (C - 1) .. 2K (C + 1): rows of P^T times the
// stiffness (STIFF) or the mass.
template <int K, typename T, bool STIFF>
__device__ __forceinline__ void restrict_matrix(const T (&f)[4 * K + 1], T (&y)[K]) {
  using CT = gen::CellTables<T, K>;
  constexpr int nf = 2 * K + 1;
#pragma unroll
  for (int a = 0; a < K; ++a) {
    T s = T(0);
    if (a == 0) {
#pragma unroll
      for (int j = 0; j < nf; ++j) s = fma(STIFF ? CT::RA[K * nf + j] : CT::RM[K * nf + j], f[j], s);
    }
#pragma unroll
    for (int j = 0; j < nf; ++j) s = fma(STIFF ? CT::RA[a * nf + j] : CT::RM[a * nf + j], f[2 * K + j], s);
    y[a] = s;
  }
}
// the same nodes of P^T f
template <int K, typename T>
__device__ __forceinline__ void restrict_values(const T (&f)[4 * K + 1], T (&y)[K]) {
  using CT = gen::CellTables<T, K>;
  constexpr int np = K + 1;
#pragma unroll
  for (int a = 0; a < K; ++a) {
    T s = a == 0 ? +f[2 * K] : T(0);
#pragma unroll
    for (int q = 1; q < 2 * K; ++q) {
      if (a == 0) s = fma(CT::P[q * np + K], f[q], s);
      if (CT::P[q * np + a] != T(0)) s = fma(CT::P[q * np + a], f[2 * K + q], s);
    }
    y[a] = s;
  }
}

// bc = P^T (b - scale A x) on the interior of the coarse level; w: the scratch.
template <int D, int K, typename T, int NT>
__device__ __forceinline__ void cycle_restrict(T* __restrict__ w, const T* __restrict__ x, const T* __restrict__ b,
                                               T* __restrict__ bc, int cells, T scale, int tid) {
  constexpr int R = 4 * K + 1;
  const int nf = 2 * K * cells + 1, nc = K * cells + 1, ci = K * cells;  // cells: coarse cells per axis
  const int lines = D == 3 ? nf * nf : nf, plane = D == 3 ? nf * nf * nc : nf * nc;
  // f <- entries 2K (C - 1) + q of a line (stride st); the cell left of the domain counts as 0
  auto fetch = [&](const T* line, int st, int C, T (&f)[R]) {
#pragma unroll
    for (int q = 0; q < R; ++q) f[q] = q < 2 * K && C == 0 ? T(0) : line[(2 * K * (C - 1) + q) * st];
  };
  T f[R], y[K], z[K];
  // x0: M x, A x, R b
  for (int t = tid; t < lines * cells; t += NT) {
    const int C = (int)((unsigned)t / (unsigned)lines), l = t - C * lines, o = l * nc + K * C;
    fetch(x + l * nf, 1, C, f);
    restrict_matrix<K, T, false>(f, y);
#pragma unroll
    for (int a = 0; a < K; ++a) w[o + a] = y[a];
    restrict_matrix<K, T, true>(f, y);
#pragma unroll
    for (int a = 0; a < K; ++a) w[plane + o + a] = y[a];
    fetch(b + l * nf, 1, C, f);
    restrict_values<K, T>(f, y);
#pragma unroll
    for (int a = 0; a < K; ++a) w[2 * plane + o + a] = y[a];
  }
  __syncthreads();
  if constexpr (D == 3) {
    // x1: M M, A M + M A, R R b
    T* w2 = w + 3 * plane;
    const int plane2 = nf * nc * nc;
    for (int t = tid; t < nf * cells * ci; t += NT) {
      const int g = (int)((unsigned)t / (unsigned)ci), c0 = t - g * ci;
      const int C = (int)((unsigned)g / (unsigned)nf), j2 = g - C * nf;
      const int i = j2 * nf * nc + c0, o = (j2 * nc + K * C) * nc + c0;
      fetch(w + i, nc, C, f);
      restrict_matrix<K, T, false>(f, y);
#pragma unroll
      for (int a = 0; a < K; ++a) w2[o + a * nc] = y[a];
      restrict_matrix<K, T, true>(f, y);
      fetch(w + plane + i, nc, C, f);
      restrict_matrix<K, T, false>(f, z);
#pragma unroll
      for (int a = 0; a < K; ++a) w2[plane2 + o + a * nc] = y[a] + z[a];
      fetch(w + 2 * plane + i, nc, C, f);
      restrict_values<K, T>(f, y);
#pragma unroll
      for (int a = 0; a < K; ++a) w2[2 * plane2 + o + a * nc] = y[a];
    }
    __syncthreads();
  }
  // the last axis: A (M M) + M (A M + M A), 2D A M + M A
  const T* in = D == 3 ? w + 3 * plane : w;
  const int step = D == 3 ? nf * nc * nc : plane, st = D == 3 ? nc * nc : nc, cols = D == 3 ? ci * ci : ci;
  for (int t = tid; t < cols * cells; t += NT) {
    const int C = (int)((unsigned)t / (unsigned)cols), r = t - C * cols;
    const int c1 = D == 3 ? (int)((unsigned)r / (unsigned)ci) : 0, i = D == 3 ? r + c1 : r;  // c1 * nc + c0
    fetch(in + i, st, C, f);
    restrict_matrix<K, T, true>(f, y);
    fetch(in + step + i, st, C, f);
    restrict_matrix<K, T, false>(f, z);
#pragma unroll
    for (int a = 0; a < K; ++a) z[a] += y[a];
    fetch(in + 2 * step + i, st, C, f);
    restrict_values<K, T>(f, y);
#pragma unroll
    for (int a = 0; a < K; ++a) bc[(K * C + a) * st + i] = fma(-scale, z[a], y[a]);
  }
  __syncthreads();
}

// x += P xc; w: the scratch.
template <int D, int K, typename T, int NT>
__device__ __forceinline__ void cycle_prolongate(T* __restrict__ w, const T* __restrict__ xc, T* __restrict__ x, int cells,
                                                 int tid) {
  using CT = gen::CellTables<T, K>;
  constexpr int np = K + 1;
  const int nf = 2 * K * cells + 1, nc = K * cells + 1, fi = nf - 1;
  const int lines = D == 3 ? nc * nc : nc;
  // fine nodes q = 0 .. 2K - 1 of a coarse cell's line from its coarse nodes
  auto expand = [&](const T (&f)[np], int q) -> T {
    T s = T(0);
#pragma unroll
    for (int a = 0; a < np; ++a)
      if (CT::P[q * np + a] != T(0)) s = fma(CT::P[q * np + a], f[a], s);
    return s;
  };
  T f[np];
  for (int t = tid; t < lines * cells; t += NT) {
    const int C = (int)((unsigned)t / (unsigned)lines), l = t - C * lines;
#pragma unroll
    for (int a = 0; a < np; ++a) f[a] = xc[l * nc + K * C + a];
#pragma unroll
    for (int q = 0; q < 2 * K; ++q) w[l * nf + 2 * K * C + q] = expand(f, q);
  }
  __syncthreads();
  const T* in = w;
  if constexpr (D == 3) {
    T* w2 = w + nc * nc * nf;
    for (int t = tid; t < nc * cells * fi; t += NT) {
      const int g = (int)((unsigned)t / (unsigned)fi), j0 = t - g * fi;
      const int C = (int)((unsigned)g / (unsigned)nc), c2 = g - C * nc;
#pragma unroll
      for (int a = 0; a < np; ++a) f[a] = w[(c2 * nc + K * C + a) * nf + j0];
#pragma unroll
      for (int q = 0; q < 2 * K; ++q) w2[(c2 * nf + 2 * K * C + q) * nf + j0] = expand(f, q);
    }
    __syncthreads();
    in = w2;
  }
  const int st = D == 3 ? nf * nf : nf, cols = D == 3 ? fi * fi : fi;
  for (int t = tid; t < cols * cells; t += NT) {
    const int C = (int)((unsigned)t / (unsigned)cols), r = t - C * cols;
    const int j1 = D == 3 ? (int)((unsigned)r / (unsigned)fi) : 0, i = D == 3 ? r + j1 : r;  // j1 * nf + j0
#pragma unroll
    for (int a = 0; a < np; ++a) f[a] = in[(K * C + a) * st + i];
#pragma unroll
    for (int q = 0; q < 2 * K; ++q) x[(2 * K * C + q) * st + i] += expand(f, q);
  }
  __syncthreads();
}

struct CycleMembers {
  const void* b[kMaxGroup];
  void* x[kMaxGroup];
  int top[kMaxGroup];
};

template <int D, int K, typename T, int TOP>
__global__ __launch_bounds__((CycleLds<D, K, T, TOP>::NT)) void cycle_kernel(CycleMembers mem, int post_reverse) {
  using C = CycleLds<D, K, T, TOP>;
  using SH = typename C::SH;
  constexpr int TEAMS = C::TEAMS, NT = C::NT, PPW = SH::PPW;
  __shared__ __align__(16) T smem[C::total];
  const int team = __builtin_amdgcn_readfirstlane((int)threadIdx.x / SH::NT), tid = threadIdx.x;
  const int top = mem.top[blockIdx.x];
  T* work = smem + C::work;
  {
    const T* b = (const T*)mem.b[blockIdx.x];
    const int o = C::offset(top), s = C::stride(top), N = C::n1d(top) * C::n1d(top) * (D == 3 ? C::n1d(top) : 1);
    for (int i = tid; i < N; i += NT) smem[o + s + i] = b[i];
  }
  // top .. 2, the coarse solve, 2 .. top
  for (int step = 0; step < 2 * top - 1; ++step) {
    const bool down = step < top;
    const int l = down ? top - step : step - top + 2;
    const int n = C::n1d(l), s = C::stride(l), half = 1 << (l - 1);
    T* x = smem + C::offset(l);
    const T* b = x + s;
    if (l == 1) {
      __syncthreads();
      double* w = reinterpret_cast<double*>(work);
      coarse_solve<D, K, T, NT>(w, w + CoarseLds<D, K>::words, b, x, tid);
      __syncthreads();
      continue;
    }
    if (down) {
      for (int i = tid; i < s; i += NT) x[i] = T(0);
      __syncthreads();
    } else {
      cycle_prolongate<D, K, T, NT>(work, smem + C::offset(l - 1), x, half, tid);
    }
    const T res_scale = D == 3 ? T(1) / T(1 << l) : T(1), sol_scale = D == 3 ? T(1 << l) : T(1);
    const bool reverse = !down && post_reverse;
    for (int ci = 0; ci < (1 << D); ++ci) {
      const int c = reverse ? (1 << D) - 1 - ci : ci;
      const int p0 = c & 1, p1 = (c >> 1) & 1, p2 = (c >> 2) & 1;
      const int cnt0 = half - p0, cnt1 = half - p1, cnt2 = D == 3 ? half - p2 : 1;
      const int groups0 = (cnt0 + PPW - 1) / PPW, blocks = groups0 * cnt1 * cnt2;
      for (int base = 0; base < blocks; base += TEAMS) {
        const int k = base + team;
        const bool active = k < blocks;
        const unsigned blk = (unsigned)(active ? k : 0);
        T* tm = work + team * C::kTeam;
        const int tt = tid - team * SH::NT;
        if constexpr (K == 1)
          colour_pass_q1<D, T, true, PPW, LdsWindow<T>>(b, x, n, p0, p1, p2, cnt0, cnt1, groups0, res_scale, sol_scale,
                                                        blk, tt, active);
        else if constexpr (D == 3)
          colour_pass_eig3<K, T, false, SH, LdsWindow<T>>(tm, b, x, n, p0, p1, p2, cnt0, cnt1, groups0, sol_scale, blk,
                                                          tt, active);
        else
          colour_pass_eig2<K, T, false, SH, LdsWindow<T>>(tm, b, x, n, p0, p1, cnt0, cnt1, groups0, sol_scale, blk, tt,
                                                          active);
        __syncthreads();
      }
    }
    if (down)
      cycle_restrict<D, K, T, NT>(work, x, b, smem + C::offset(l - 1) + C::stride(l - 1), half, res_scale, tid);
  }
  T* xo = (T*)mem.x[blockIdx.x];
  const int o = C::offset(top), N = C::n1d(top) * C::n1d(top) * (D == 3 ? C::n1d(top) : 1);
  for (int i = tid; i < N; i += NT) xo[i] = smem[o + i];
}

// ------------------------------------------------------------------ host side

// Patch grid of one colour on one level: parities, counts per axis, workgroups along x0.
template <int D, int K>
struct ColourGrid {
  int p[3] = {0, 0, 0}, cnt[3] = {1, 1, 1};
  int groups0 = 0;
  long long blocks = 0;
  bool ok = true;  // the 32-bit block (byte) offsets of the kernel are valid
  ColourGrid(const LevelGeom& g, int colour, int PPW = SmootherShape<D, K>::PPW) {
    const int half = (int)(g.ncells / 2);
    for (int a = 0; a < D; ++a) {
      p[a] = (colour >> a) & 1;
      cnt[a] = half - p[a];
    }
    for (int a = 0; a < D; ++a)
      if (cnt[a] <= 0) return;  // empty colour (coarsest level)
    groups0 = (cnt[0] + PPW - 1) / PPW;
    blocks = (long long)groups0 * cnt[1] * (D == 3 ? cnt[2] : 1);
    constexpr long long n = 2 * K + 1;
    const long long span = (D == 3 ? (n - 1) * g.n1d * g.n1d : 0) + (n - 1) * g.n1d + 2 * K * PPW + 1;
    ok = blocks <= 0x7fffffffLL && span < (1LL << 29);  // byte offsets of 8-byte words fit in 32 bits
  }
};

template <int D, int K, typename T, int MODE, typename SH>
static hipError_t launch_shape(const LevelGeom& g, const ColourGrid<D, K>& cg, const void* b, void* x,
                               hipStream_t st) {
  // Abar_h = h^(d-2) Abar_1 ; A_j,h^{-1} = h^(2-d) A_j,1^{-1}
  const T res_scale = (T)(D == 3 ? g.h : 1.0);
  const T sol_scale = (T)(D == 3 ? 1.0 / g.h : 1.0);
  hipLaunchKernelGGL((colour_pass_kernel<D, K, T, MODE, SH>), dim3((unsigned)cg.blocks), dim3(SH::NT), 0, st,
                     (const T*)b, (T*)x, g.n1d, cg.p[0], cg.p[1], cg.p[2], cg.cnt[0], cg.cnt[1], cg.groups0,
                     res_scale, sol_scale);
  return hipGetLastError();
}

// Shapes of a mode: the large one, and the small-launch one a launch takes when the large one would
// give fewer than kMinBlocks workgroups.
template <int D, int K, typename T, int MODE>
struct ModeShapes {
  using Large = LineShape<SmootherShape<D, K>::PPW, SmootherShape<D, K>::NT>;
  using Small = LineShape<LatencyPPW<D, K>::value, SmootherShape<D, K>::NT>;
  static constexpr long long kMinBlocks = kLatencyBlocks;
};
template <int D, int K, typename T>
struct ModeShapes<D, K, T, kModeMultiplicative> {
  using Large = typename EigShapes<D, K, T>::Large;
  using Small = typename EigShapes<D, K, T>::Small;
  static constexpr long long kMinBlocks = kEigWaves * 64 / Large::NT;
};
template <int D, int K, typename T>
struct ModeShapes<D, K, T, kModeBoundary> : ModeShapes<D, K, T, kModeMultiplicative> {};
template <int D, int K, typename T>
struct ModeShapes<D, K, T, kModeAdditive> {
  using Large = typename AddShapes<D, K, T>::Large;
  using Small = typename AddShapes<D, K, T>::Small;
  static constexpr long long kMinBlocks = kEigWaves * 64 / Large::NT;
};
template <int D, int K, typename T>
struct ModeShapes<D, K, T, kModeZero> : ModeShapes<D, K, T, kModeAdditive> {};
using WideShape = LineShape<kWidePPW, kWideNT>;
using MfmaShape = LineShape<kMfmaPPW, 256>;

// The wide shape's launch: enough workgroups to leave the small-launch regime and few idle patch
// slots at row ends.
template <int D, int K>
static bool wide_fits(const ColourGrid<D, K>& cw) {
  return cw.ok && cw.blocks >= kLatencyBlocks &&
         (double)(cw.groups0 * kWidePPW - cw.cnt[0]) <= kWideIdle * (double)cw.cnt[0];
}

// True when a pass of this colour and level runs the matrix-core form: its launch has at least
// kLatencyBlocks workgroups.  A packed launch must give each member the arithmetic of its stand-alone
// pass, so that a result does not depend on the requests it is served with.
template <int D, int K>
static bool mfma_fits(const LevelGeom& g, int colour) {
  return ColourGrid<D, K>(g, colour, kMfmaPPW).blocks >= kLatencyBlocks;
}

template <int D, int K, typename T, int MODE>
static hipError_t launch_one(const LevelGeom& g, int colour, const void* b, void* x, hipStream_t st) {
  using Large = typename ModeShapes<D, K, T, MODE>::Large;
  using Small = typename ModeShapes<D, K, T, MODE>::Small;
  if constexpr (HasWideForm<D, K, T, MODE>::value) {
    const ColourGrid<D, K> cw(g, colour, kWidePPW);
    if (wide_fits(cw)) return launch_shape<D, K, T, MODE, WideShape>(g, cw, b, x, st);
  }
  if constexpr (MODE == kModeMultiplicative || MODE == kModeBoundary) {
    using Far = typename FarShape<D, K, T>::type;
    if constexpr (!std::is_void<Far>::value) {
      const ColourGrid<D, K> cf(g, colour, Far::PPW);
      if (cf.ok && 2.0 * sizeof(T) * std::pow((double)g.n1d, D) > (double)kLastLevelCache)
        return launch_shape<D, K, T, MODE, Far>(g, cf, b, x, st);
    }
  }
  const ColourGrid<D, K> cg(g, colour, Large::PPW);
  if (!cg.ok) return hipErrorInvalidConfiguration;
  if (cg.blocks == 0) return hipSuccess;
  if constexpr (!std::is_same<Small, Large>::value) {
    if (cg.blocks < ModeShapes<D, K, T, MODE>::kMinBlocks) {
      const ColourGrid<D, K> cl(g, colour, Small::PPW);
      if (!cl.ok) return hipErrorInvalidConfiguration;
      return launch_shape<D, K, T, MODE, Small>(g, cl, b, x, st);
    }
  }
  return launch_shape<D, K, T, MODE, Large>(g, cg, b, x, st);
}

// One launch per kMaxGroup of the members that `take` accepts, in workgroups of shape SH.
template <int D, int K, typename T, int MODE, typename SH, typename F>
static hipError_t launch_group_shape(int colour, const ColourPassMember* mem, int nm, hipStream_t st, F take) {
  ColourPassGroup grp;
  grp.n = 0;
  long long total = 0;
  auto flush = [&]() -> hipError_t {
    if (grp.n == 0) return hipSuccess;
    hipLaunchKernelGGL((colour_pass_group_kernel<D, K, T, MODE, SH>), dim3((unsigned)total), dim3(SH::NT), 0, st, grp);
    grp.n = 0;
    total = 0;
    return hipGetLastError();
  };
  for (int i = 0; i < nm; ++i) {
    if (!take(mem[i].g)) continue;
    const ColourGrid<D, K> cg(mem[i].g, colour, SH::PPW);
    if (!cg.ok) return hipErrorInvalidConfiguration;
    if (cg.blocks == 0) continue;
    if (grp.n == kMaxGroup || total + cg.blocks > 0x7fffffffLL) {
      hipError_t e = flush();
      if (e != hipSuccess) return e;
    }
    ColourPassDesc& d = grp.e[grp.n++];
    d.b = mem[i].b;
    d.x = mem[i].x;
    d.n1d = mem[i].g.n1d;
    d.p[0] = cg.p[0];
    d.p[1] = cg.p[1];
    d.p[2] = cg.p[2];
    d.cnt0 = cg.cnt[0];
    d.cnt1 = cg.cnt[1];
    d.groups0 = cg.groups0;
    d.block_begin = (int)total;
    d.res_scale = D == 3 ? mem[i].g.h : 1.0;
    d.sol_scale = D == 3 ? 1.0 / mem[i].g.h : 1.0;
    total += cg.blocks;
  }
  return flush();
}

// The members that `take` accepts: the small-launch shape when all of them together would give fewer
// than kMinBlocks workgroups of the large one (the shapes give the same values bit for bit).
template <int D, int K, typename T, int MODE, typename F>
static hipError_t launch_group(int colour, const ColourPassMember* mem, int nm, hipStream_t st, F take) {
  using Large = typename ModeShapes<D, K, T, MODE>::Large;
  using Small = typename ModeShapes<D, K, T, MODE>::Small;
  long long blocks = 0;
  for (int i = 0; i < nm; ++i)
    if (take(mem[i].g)) blocks += ColourGrid<D, K>(mem[i].g, colour, Large::PPW).blocks;
  if (blocks < ModeShapes<D, K, T, MODE>::kMinBlocks)
    return launch_group_shape<D, K, T, MODE, Small>(colour, mem, nm, st, take);
  return launch_group_shape<D, K, T, MODE, Large>(colour, mem, nm, st, take);
}

// The kernel of kModeTail: the eigenbasis form without the loads of x^I, which gives the same values, where
// the multiplicative pass has that form, else the multiplicative pass itself.
template <typename T>
constexpr int kPrec = sizeof(T) == 8 ? 0 : 1;
template <int D, int K, typename T>
struct HasEigenForm {
  static constexpr bool value = K >= (D == 2 && sizeof(T) == 4 ? 5 : 3);  // has_eigen_form
};
template <int D, int K, typename T>
constexpr int tail_mode() {
  return HasEigenForm<D, K, T>::value ? kModeBoundary : K == 1 ? kModeMultiplicative : kModeResidual;
}

template <int D, int K, typename T>
static hipError_t dispatch_mode(const LevelGeom& g, int mode, int colour, const void* b, void* x, hipStream_t st) {
  switch (mode) {
    case kModeMultiplicative:
      if constexpr (HasEigenForm<D, K, T>::value || K == 1)
        if (K == 1 || eigen_step_fits(g, kPrec<T>)) return launch_one<D, K, T, kModeMultiplicative>(g, colour, b, x, st);
      return dispatch_mode<D, K, T>(g, kModeResidual, colour, b, x, st);
    case kModeAdditive: return launch_one<D, K, T, kModeAdditive>(g, colour, b, x, st);
    case kModeTail: return launch_one<D, K, T, tail_mode<D, K, T>()>(g, colour, b, x, st);
    case kModeResidual:
      return launch_one<D, K, T, K == 1 ? kModeMultiplicative : kModeResidual>(g, colour, b, x, st);
    case kModeBoundary: return launch_one<D, K, T, kModeBoundary>(g, colour, b, x, st);
    case kModeMfma:
      if constexpr (HasMfmaForm<D, K, T>::value) {
        const ColourGrid<D, K> cm(g, colour, kMfmaPPW);
        if (!cm.ok) return hipErrorInvalidConfiguration;
        if (mfma_fits<D, K>(g, colour)) return launch_shape<D, K, T, kModeMfma, MfmaShape>(g, cm, b, x, st);
      }
      return dispatch_mode<D, K, T>(g, kModeMultiplicative, colour, b, x, st);
    case kModeZero:
      if (colour != 0) return hipErrorInvalidValue;  // only colour 0's closures tile the grid
      return launch_one<D, K, T, kModeZero>(g, colour, b, x, st);
  }
  return hipErrorInvalidValue;
}

template <int D, int K>
static hipError_t dispatch_prec(const LevelGeom& g, int prec, int mode, int colour, const void* b, void* x,
                                hipStream_t st) {
  return prec == 0 ? dispatch_mode<D, K, double>(g, mode, colour, b, x, st)
                   : dispatch_mode<D, K, float>(g, mode, colour, b, x, st);
}

template <int D>
static hipError_t dispatch_k(const LevelGeom& g, int prec, int mode, int colour, const void* b, void* x,
                             hipStream_t st) {
  switch (g.k) {
    case 1: return dispatch_prec<D, 1>(g, prec, mode, colour, b, x, st);
    case 2: return dispatch_prec<D, 2>(g, prec, mode, colour, b, x, st);
    case 3: return dispatch_prec<D, 3>(g, prec, mode, colour, b, x, st);
    case 4: return dispatch_prec<D, 4>(g, prec, mode, colour, b, x, st);
    case 5: return dispatch_prec<D, 5>(g, prec, mode, colour, b, x, st);
    case 6: return dispatch_prec<D, 6>(g, prec, mode, colour, b, x, st);
    case 7: return dispatch_prec<D, 7>(g, prec, mode, colour, b, x, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_colour_pass(const LevelGeom& g, int prec, int mode, int colour, const void* b, void* x,
                              hipStream_t st) {
  return g.dim == 2 ? dispatch_k<2>(g, prec, mode, colour, b, x, st) : dispatch_k<3>(g, prec, mode, colour, b, x, st);
}

template <int D, int K, typename T>
static hipError_t group_mode(int mode, int colour, const ColourPassMember* m, int nm, hipStream_t st) {
  auto all = [](const LevelGeom&) { return true; };
  switch (mode) {
    case kModeMultiplicative:
    case kModeResidual: {
      auto eig = [mode](const LevelGeom& g) { return K == 1 || (mode == kModeMultiplicative && eigen_step_fits(g, kPrec<T>)); };
      hipError_t e = hipSuccess;
      if constexpr (HasEigenForm<D, K, T>::value || K == 1) e = launch_group<D, K, T, kModeMultiplicative>(colour, m, nm, st, eig);
      if (e != hipSuccess) return e;
      if constexpr (K > 1)
        return launch_group<D, K, T, kModeResidual>(colour, m, nm, st, [&](const LevelGeom& g) { return !eig(g); });
      return e;
    }
    case kModeAdditive: return launch_group<D, K, T, kModeAdditive>(colour, m, nm, st, all);
    case kModeTail: return launch_group<D, K, T, tail_mode<D, K, T>()>(colour, m, nm, st, all);
    case kModeBoundary: return launch_group<D, K, T, kModeBoundary>(colour, m, nm, st, all);
    case kModeZero:
      if (colour != 0) return hipErrorInvalidValue;
      return launch_group<D, K, T, kModeZero>(colour, m, nm, st, all);
    case kModeMfma: {
      // the members whose own pass runs on the matrix cores, then the others as kModeMultiplicative
      std::vector<ColourPassMember> rest;
      if constexpr (HasMfmaForm<D, K, T>::value) {
        auto fits = [colour](const LevelGeom& g) { return mfma_fits<D, K>(g, colour); };
        hipError_t e = launch_group_shape<D, K, T, kModeMfma, MfmaShape>(colour, m, nm, st, fits);
        if (e != hipSuccess) return e;
        for (int i = 0; i < nm; ++i)
          if (!fits(m[i].g)) rest.push_back(m[i]);
      } else {
        rest.assign(m, m + nm);
      }
      return group_mode<D, K, T>(kModeMultiplicative, colour, rest.data(), (int)rest.size(), st);
    }
  }
  return hipErrorInvalidValue;
}

template <int D, int K>
static hipError_t group_prec(int prec, int mode, int colour, const ColourPassMember* m, int nm, hipStream_t st) {
  return prec == 0 ? group_mode<D, K, double>(mode, colour, m, nm, st)
                   : group_mode<D, K, float>(mode, colour, m, nm, st);
}

template <int D>
static hipError_t group_k(int k, int prec, int mode, int colour, const ColourPassMember* m, int nm, hipStream_t st) {
  switch (k) {
    case 1: return group_prec<D, 1>(prec, mode, colour, m, nm, st);
    case 2: return group_prec<D, 2>(prec, mode, colour, m, nm, st);
    case 3: return group_prec<D, 3>(prec, mode, colour, m, nm, st);
    case 4: return group_prec<D, 4>(prec, mode, colour, m, nm, st);
    case 5: return group_prec<D, 5>(prec, mode, colour, m, nm, st);
    case 6: return group_prec<D, 6>(prec, mode, colour, m, nm, st);
    case 7: return group_prec<D, 7>(prec, mode, colour, m, nm, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_colour_pass_group(int dim, int k, int prec, int mode, int colour, const ColourPassMember* members,
                                    int n_members, hipStream_t st) {
  return dim == 2 ? group_k<2>(k, prec, mode, colour, members, n_members, st)
                  : group_k<3>(k, prec, mode, colour, members, n_members, st);
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

template <int D, int K, typename T>
static hipError_t coarse_fused(const ColourPassMember* mem, int nm, hipStream_t st) {
  for (int i0 = 0; i0 < nm; i0 += kMaxGroup) {
    const int n = nm - i0 < kMaxGroup ? nm - i0 : kMaxGroup;
    FusedMembers fm{};
    for (int i = 0; i < n; ++i) {
      fm.b[i] = mem[i0 + i].b;
      fm.x[i] = mem[i0 + i].x;
    }
    hipLaunchKernelGGL((coarse_solve_kernel<D, K, T>), dim3(n), dim3(256), 0, st, fm);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
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

// The highest level of cycle_kernel per (dim, degree, precision): 1 where one workgroup loses to the launches it
// saves or its LDS does not suffice.  Four CG iterations with the cycle on the level as preconditioner, us, with the
// cycle up to the level below against up to it: 2D degree 1 level 5 401 / 318, level 6 428 / 401; degree 2 level 4
// FP32 381 / 347, level 5 476 / 541 (not taken); degree 3 level 4 FP32 485 / 455, FP64 518 / 528 (not taken); degree
// 4 level 3 388 / 325, level 4 475 / 560 (not taken); degree 7 level 3 FP32 520 / 450, FP64 687 / 688.  3D degree 1
// level 3 FP32 487 / 455, FP64 485 / 501 (not taken); degree 2 level 2 429 / 341, level 3 621 / 749 (not taken);
// degree 3 level 2 494 / 390, FP64 545 / 440; degree 4 level 2 FP32 563 / 458.
template <int D, int K, typename T>
struct CycleTop {
  static constexpr bool f32 = sizeof(T) == 4;
  static constexpr int value = D == 2 ? (K == 1 ? 6 : K == 2 ? 4 : K == 3 && f32 ? 4 : 3)
                                      : (K == 1 ? (f32 ? 3 : 2) : K <= 3 || (K == 4 && f32) ? 2 : 1);
};

int cycle_top(int dim, int k, int prec) {
  int top = 1;
  (void)with_degree(dim, k, [&](auto d, auto kk) {
    constexpr int D = decltype(d)::value, K = decltype(kk)::value;
    top = prec == 0 ? CycleTop<D, K, double>::value : CycleTop<D, K, float>::value;
    return hipSuccess;
  });
  return top;
}

template <int D, int K, typename T>
static hipError_t cycle_launch(const ColourPassMember* mem, int nm, bool post_reverse, hipStream_t st) {
  constexpr int TOP = CycleTop<D, K, T>::value;
  if constexpr (TOP < 2) {
    return hipErrorInvalidValue;
  } else {
    for (int i0 = 0; i0 < nm; i0 += kMaxGroup) {
      const int n = nm - i0 < kMaxGroup ? nm - i0 : kMaxGroup;
      CycleMembers cm{};
      for (int i = 0; i < n; ++i) {
        if (mem[i0 + i].g.level < 1 || mem[i0 + i].g.level > TOP) return hipErrorInvalidValue;
        cm.b[i] = mem[i0 + i].b;
        cm.x[i] = mem[i0 + i].x;
        cm.top[i] = mem[i0 + i].g.level;
      }
      hipLaunchKernelGGL((cycle_kernel<D, K, T, TOP>), dim3(n), dim3(CycleLds<D, K, T, TOP>::NT), 0, st, cm,
                         post_reverse ? 1 : 0);
      hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
}

hipError_t launch_cycle(int dim, int k, int prec, bool post_reverse, const ColourPassMember* mem, int nm,
                        hipStream_t st) {
  return with_degree(dim, k, [&](auto d, auto kk) {
    constexpr int D = decltype(d)::value, K = decltype(kk)::value;
    return prec == 0 ? cycle_launch<D, K, double>(mem, nm, post_reverse, st)
                     : cycle_launch<D, K, float>(mem, nm, post_reverse, st);
  });
}

// Spans from level 2 up, [dim - 2][k - 1][prec], where a fused step takes less device time than its single passes,
// or up to 10% more (it also saves the host 2.4 us per launch).  One step, us, single passes against fused, FP32 /
// FP64: 3D degree 1 levels 2-4 17-20 / 18-22 against 10-15; degree 2 22, 25, 25 against 19, 24, 26; degree 3 30, 31,
// 31 against 23, 29, 34; degree 4 level 2 32 / 38 against 28 / 39, level 4 36 / 44 against 43 / 58 (not taken: a
// workgroup runs on one compute unit, and four teams saturate its vector units); degree 7 level 2 47 / 66 against
// 62 / 129.  2D degree 1 levels 2-6 6.6-9.5 against 3.4-5.8; degree 4 level 3 12 / 15 against 9.5 / 14, level 5
// 13.9 / 15.6 against 11.9 / 16.8; degree 7 level 3 16 / 22 against 14 / 21, level 5 FP64 23 against 28.  Levels up
// to cycle_top() serve the additive step only (corrections there run in the cycle's launch).
static const char* const kFusedSpans[2][7][2] = {
    {{"222111", "222111"},  // 2D; {FP64, FP32}
     {"222111", "222111"},
     {"2211", "22111"},
     {"2211", "2211"},
     {"221", "2211"},
     {"211", "2211"},
     {"111", "2211"}},
    {{"321", "321"},  // 3D
     {"321", "321"},
     {"31", "311"},
     {"3", "31"},
     {"", "3"},
     {"", "1"},
     {"", ""}}};

// The additive step's teams hold more registers: in FP64 from 2D degree 5 up they run at 3.2-5.5 us per pass on levels
// 2-4 against 2.9-4.6 of its single passes, in FP32 from degree 5 up on level 5 at 2.8-4.0 against 2.9-3.6.
int fused_span(const LevelGeom& g, int prec, bool additive) {
  if (additive && g.dim == 2 && g.k >= 5 && (prec == 0 || g.level > 4)) return 0;
  const char* s = kFusedSpans[g.dim - 2][g.k - 1][prec];
  for (int i = 2; *s; ++i, ++s)
    if (i == g.level) return *s - '0';
  return 0;
}

hipError_t launch_smooth_fused(const LevelGeom& g, int prec, bool additive, int span, bool reverse, bool clear,
                               const ColourPassMember* mem, int nm, hipStream_t st) {
  return with_degree(g.dim, g.k, [&](auto d, auto k) {
    constexpr int D = decltype(d)::value, K = decltype(k)::value;
    if (additive)
      return prec == 0 ? smooth_fused<D, K, double, true>(g, span, reverse, clear, mem, nm, st)
                       : smooth_fused<D, K, float, true>(g, span, reverse, clear, mem, nm, st);
    return prec == 0 ? smooth_fused<D, K, double, false>(g, span, reverse, clear, mem, nm, st)
                     : smooth_fused<D, K, float, false>(g, span, reverse, clear, mem, nm, st);
  });
}

hipError_t launch_coarse_solve(int dim, int k, int prec, const ColourPassMember* mem, int nm, hipStream_t st) {
  return with_degree(dim, k, [&](auto d, auto kk) {
    constexpr int D = decltype(d)::value, K = decltype(kk)::value;
    return prec == 0 ? coarse_fused<D, K, double>(mem, nm, st) : coarse_fused<D, K, float>(mem, nm, st);
  });
}

// ------------------------------------------------------------ host-side launch geometry

namespace {

// Every workgroup of one colour's launch with PPW patches per workgroup: its patches lie in the
// colour and inside the grid, the workgroups cover the colour's patches once, and the farthest
// closure node of a workgroup is within the kernels' 32-bit byte offsets (8-byte words).
template <int D, int K, int PPW>
bool colour_shape_ok(const LevelGeom& g, int colour, long long* nblk, std::string* why) {
  const ColourGrid<D, K> cg(g, colour, PPW);
  if (cg.blocks == 0) return true;
  const std::string tag = "colour " + std::to_string(colour) + ", " + std::to_string(PPW) + " patches per workgroup: ";
  if (!cg.ok) return *why = tag + "launch refused (offsets or grid beyond 32 bits)", false;
  const long long n1d = g.n1d, nc = g.ncells, span = 2LL * K;
  long long patches = 0;
  for (long long b = 0; b < cg.blocks; ++b) {
    const ColourBlock cb = colour_block<D, K, PPW>((unsigned)b, cg.p[0], cg.p[1], cg.p[2], cg.cnt[0], cg.cnt[1],
                                                   cg.groups0);
    if (cb.count < 1 || cb.count > PPW) return *why = tag + "workgroup without patches", false;
    const long long s[3] = {cb.s0, cb.s1, cb.s2};
    for (int a = 0; a < D; ++a) {
      const long long v = s[a] / K + 1;  // vertex of the workgroup's first patch
      if (s[a] % K != 0 || v < 1 || v > nc - 1 || ((v - 1) & 1) != cg.p[a])
        return *why = tag + "patch outside the colour", false;
    }
    if (s[0] / K + 1 + 2LL * (cb.count - 1) > nc - 1) return *why = tag + "patch past the last vertex", false;
    if (cb.s0 + span * cb.count > n1d - 1 || cb.s1 + span > n1d - 1 || (D == 3 && cb.s2 + span > n1d - 1))
      return *why = tag + "closure outside the grid", false;
    const long long far = (D == 3 ? span * n1d * n1d : 0) + span * n1d + span * cb.count;
    if (far * 8 >= (1LL << 32)) return *why = tag + "closure offsets beyond 32 bits", false;
    patches += cb.count;
  }
  const long long want = (long long)cg.cnt[0] * cg.cnt[1] * (D == 3 ? cg.cnt[2] : 1);
  if (patches != want) return *why = tag + "workgroups do not cover the colour once", false;
  *nblk += cg.blocks;
  return true;
}

template <int D, int K>
bool colour_launches_ok(const LevelGeom& g, long long* nblk, std::string* why) {
  for (int c = 0; c < (1 << D); ++c) {
    if (!colour_shape_ok<D, K, SmootherShape<D, K>::PPW>(g, c, nblk, why)) return false;
    if (!colour_shape_ok<D, K, LatencyPPW<D, K>::value>(g, c, nblk, why)) return false;
    if constexpr (HasMfmaForm<D, K, float>::value)
      if (!colour_shape_ok<D, K, kMfmaPPW>(g, c, nblk, why)) return false;
    if (!colour_shape_ok<D, K, AddShapes<D, K, float>::Large::PPW>(g, c, nblk, why)) return false;
    if (!colour_shape_ok<D, K, AddShapes<D, K, float>::Small::PPW>(g, c, nblk, why)) return false;
    if (!colour_shape_ok<D, K, EigShapes<D, K, float>::Large::PPW>(g, c, nblk, why)) return false;
    if (!colour_shape_ok<D, K, EigShapes<D, K, float>::Small::PPW>(g, c, nblk, why)) return false;
    if (!colour_shape_ok<D, K, EigShapes<D, K, double>::Large::PPW>(g, c, nblk, why)) return false;
    if (!colour_shape_ok<D, K, EigShapes<D, K, double>::Small::PPW>(g, c, nblk, why)) return false;
    if constexpr (!std::is_void<typename FarShape<D, K, float>::type>::value)
      if (!colour_shape_ok<D, K, FarShape<D, K, float>::type::PPW>(g, c, nblk, why)) return false;
    if constexpr (HasWideForm<D, K, float, kModeResidual>::value)
      if (!colour_shape_ok<D, K, kWidePPW>(g, c, nblk, why)) return false;
  }
  return true;
}

}  // namespace

bool check_colour_launches(const LevelGeom& g, long long* blocks, std::string* why) {
  switch (g.dim * 10 + g.k) {
    case 21: return colour_launches_ok<2, 1>(g, blocks, why);
    case 22: return colour_launches_ok<2, 2>(g, blocks, why);
    case 23: return colour_launches_ok<2, 3>(g, blocks, why);
    case 24: return colour_launches_ok<2, 4>(g, blocks, why);
    case 25: return colour_launches_ok<2, 5>(g, blocks, why);
    case 26: return colour_launches_ok<2, 6>(g, blocks, why);
    case 27: return colour_launches_ok<2, 7>(g, blocks, why);
    case 31: return colour_launches_ok<3, 1>(g, blocks, why);
    case 32: return colour_launches_ok<3, 2>(g, blocks, why);
    case 33: return colour_launches_ok<3, 3>(g, blocks, why);
    case 34: return colour_launches_ok<3, 4>(g, blocks, why);
    case 35: return colour_launches_ok<3, 5>(g, blocks, why);
    case 36: return colour_launches_ok<3, 6>(g, blocks, why);
    case 37: return colour_launches_ok<3, 7>(g, blocks, why);
  }
  *why = "unsupported (dim, degree)";
  return false;
}

hipError_t init_smoother_tables() {
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
