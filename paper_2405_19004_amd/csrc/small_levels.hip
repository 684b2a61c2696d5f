// Kernels of the small levels, where launches cost more than the work in them: several colours of a smoothing step in
// one launch, the coarse solve, and the small levels of a V-cycle in one launch.
// They loop over colours and levels around unrolled passes, so this file is compiled without machine-code loop
// invariant motion: hoisted out of those loops the FP64 table constants (two scalar registers each) spilled by the
// hundred (cycle_kernel 2D degrees 4-7 FP64: 400-1500 spills; without, 18-91, and four CG iterations on level 3 in
// 337-558 us against 358-650).  The additive step's fused form measured 4-8% slower that way and stays in smoother.hip.
#include "colour_pass.hpp"

namespace vps {

hipError_t init_small_level_tables() { return upload_tables(); }

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
  static constexpr int kTeam = team_lds<D, K, SH, false>();
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
  if (additive) return launch_additive_fused(g, prec, span, reverse, clear, mem, nm, st);
  return with_degree(g.dim, g.k, [&](auto d, auto k) {
    constexpr int D = decltype(d)::value, K = decltype(k)::value;
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

}  // namespace vps
