// Launch functions of the device code (HIP translation units), called by the
// host-side library.  All launches are asynchronous on the given stream and
// return the launch status.
#pragma once
#include <hip/hip_runtime.h>

#include <string>

#include "device_common.hpp"

namespace vps {

// Scalar slots of the CG scalar block (device memory, doubles).
enum : int {
  kScRZ = 0,     // r.z of the current iterate
  kScPQ = 10,    // p.A p                         (written together with slot 11)
  kScRR = 2,     // r.r after the update          (written together with kScRZOld)
  kScRZOld = 3,  // r_new . z_old (flexible beta)
  kScRZNew = 4,  // r_new . z_new
  kScBB = 7,     // b.b
  kScTrue = 8,   // true residual norm squared    (written together with kScAux2)
  kScAux2 = 9,
  kScCount = 16
};

hipError_t init_smoother_tables();     // smoother.hip, and through it
hipError_t init_small_level_tables();  // small_levels.hip

// Colour-pass kernels: multiplicative (residual, then x^I += A_j^{-1} r), additive
// (x^I += A_j^{-1} b^I) and Boundary (x^I = A_j^{-1} (b^I - A^{IB} x^B), x^I never read).
// kModeMfma: the multiplicative pass with the residual contractions on the matrix cores (3D Q4
// FP32, default launch shape); elsewhere the same as kModeMultiplicative.
// kModeZero: colour 0 of the multiplicative pass on a zero iterate, x <- S_0(0, b): writes
// A_j^{-1} b^I on the colour's patch interiors and 0 on every other node (the closures of colour 0
// tile the grid), so x need not be cleared first and is never read.
// The multiplicative pass has two forms (smoother.hip).  The eigenbasis form is faster; its rounding is
// relative to the variation of x over a patch, a white error.  The residual form x + A_j^{-1} (b - A x)
// rounds a residual, a smooth error: iterated to stagnation it reaches a lower residual.  So:
// kModeMultiplicative: one step on a caller's iterate.  Eigenbasis form where eigen_step_fits (there its
//   error against FP64 is the smaller one), and a patch with a non-finite old value becomes non-finite;
//   elsewhere the residual form.
// kModeTail: the eigenbasis form without looking at old interior values, for corrections (V-cycle levels
//   that start from 0: the rounding is relative to the correction) and for later colours of a step whose
//   first colour was 0.  After colour 0, whose closures tile the grid, the non-finite values are a union
//   of whole patch interiors, and every other patch that overlaps one has it on its closure's rim too:
//   the values are those of kModeMultiplicative.
// kModeResidual: the residual form, for the last smoothing step of a V-cycle on a caller's iterate, which
//   decides how far repeated V-cycles reduce the residual.
enum { kModeMultiplicative = 0, kModeAdditive = 1, kModeBoundary = 2, kModeMfma = 4, kModeZero = 5, kModeTail = 6, kModeResidual = 7 };

// The eigenbasis form serves degrees 3-7, in 2D FP32 degrees 5-7: degree 1 is a stencil, and below these the
// face transforms cost what they save (finest pass against the residual form, us: 3D degree 2, 256^3 cells,
// FP32 41.0 / 41.5, FP64 61.2 / 61.7; 2D 2048^2 cells degree 2 34.2 / 31.3 and 55.2 / 56.2; 2D 1024^2 FP32
// degree 3 20.7 / 19.8, degree 4 36.5 / 33.7).
inline bool has_eigen_form(int dim, int k, int prec) { return k >= (dim == 2 && prec == 1 ? 5 : 3); }
// For single steps, 3D levels with fewer than 16 cells per axis keep the residual form as well: a patch spans a
// quarter of the domain or more there, and the eigenbasis form's error (FP32 model, one step, degree 4) is
// 1.5 times the residual form's on 8^3 cells, 0.8 times on 16^3; in 2D it is 0.05-0.6 times.
inline bool eigen_step_fits(const LevelGeom& g, int prec) {
  return has_eigen_form(g.dim, g.k, prec) && (g.dim == 2 || g.level >= 4);
}

// One member of a packed colour-pass launch (see launch_colour_pass_group).
struct ColourPassDesc {
  const void* b;
  void* x;
  long long n1d;
  int p[3];
  int cnt0, cnt1, groups0;
  int block_begin;
  double res_scale, sol_scale;
};
constexpr int kMaxGroup = 16;
struct ColourPassGroup {
  int n;
  ColourPassDesc e[kMaxGroup];
};
struct ColourPassMember {
  LevelGeom g;
  const void* b;
  void* x;
};
// Colour `colour` on every member (same dim, degree and precision; any levels) with one launch
// per kMaxGroup members.  Each member's arithmetic is exactly that of launch_colour_pass.
hipError_t launch_colour_pass_group(int dim, int k, int prec, int mode, int colour,
                                    const ColourPassMember* members, int n_members, hipStream_t st);

// One smoothing step of corrections (the eigenbasis form without a look at old interior values; ascending colours, or
// descending with reverse), or an additive step, on the members, all on the level g, several colours per launch.
// span (1..dim): the unit of one workgroup (1: a row of patches along x0, with the two colours that differ in its
// parity; dim: the grid, all colours).  clear (ascending only): x holds anything and counts as 0.
hipError_t launch_smooth_fused(const LevelGeom& g, int prec, bool additive, int span, bool reverse, bool clear,
                               const ColourPassMember* members, int n_members, hipStream_t st);
hipError_t launch_additive_fused(const LevelGeom& g, int prec, int span, bool reverse, bool clear,
                                 const ColourPassMember* members, int n_members, hipStream_t st);
// The span of a step on a level; 0: one colour per launch.
int fused_span(const LevelGeom& g, int prec, bool additive);
// x = A_1^{-1} b on level 1 for every member, in FP64 arithmetic.
hipError_t launch_coarse_solve(int dim, int k, int prec, const ColourPassMember* members, int n_members,
                               hipStream_t st);
// x = V-cycle of b from x = 0 (multiplicative smoother; x holds anything on entry) on every member's level g.level,
// in one launch; levels up to cycle_top(), which is 1 where there is no such form.
int cycle_top(int dim, int k, int prec);
hipError_t launch_cycle(int dim, int k, int prec, bool post_reverse, const ColourPassMember* members, int n_members,
                        hipStream_t st);

// smoother.hip
hipError_t launch_colour_pass(const LevelGeom& g, int prec, int mode, int colour, const void* b, void* x,
                              hipStream_t st);

// grid.hip (interior outputs only)
hipError_t launch_operator(const LevelGeom& g, int prec, const void* x, const void* b_or_null, void* y, hipStream_t st);
// Per-workgroup partial sums the two fused operator forms below take on level g (0: no fused
// form on that level).
long long fused_reduction_parts(const LevelGeom& g);
// q = A p in FP64 with the partials of p.q per workgroup (at most max_parts) in part and, when out is not null, out[0] =
// their sum in a fixed order; *fused = false (nothing launched) where that form is not available.
hipError_t launch_operator_pq(const LevelGeom& g, const double* p, double* q, double* part, long long max_parts,
                              double* out, hipStream_t st, bool* fused);
// out[0] = |b - A x|^2 (interior, FP64) summed in a fixed order from per-workgroup partials, the
// residual itself not stored; *fused = false (nothing launched) where that form is not available.
hipError_t launch_residual_norm2(const LevelGeom& g, const double* x, const double* b, double* part,
                                 long long max_parts, double* out, hipStream_t st, bool* fused, double* host);
// Restriction P^T of a fine-level vector (fine boundary entries ignored, coarse boundary written 0);
// t is scratch of restrict_scratch_elems(fine) elements (none in 2D: one kernel, no intermediate).
hipError_t launch_restrict(const LevelGeom& fine, int prec, const void* rf, void* rc, void* t, hipStream_t st);
inline long long restrict_scratch_elems(int dim, int k, int fine_level) {
  const long long nf = (long long)k * (1LL << fine_level) + 1, nc = (long long)k * (1LL << (fine_level - 1)) + 1;
  return dim == 2 ? 0 : nf * nc * nc;
}
hipError_t launch_prolongate_add(const LevelGeom& fine, int prec, const void* e, void* xf, hipStream_t st);
// The allocation-free restriction's scratch: a static device array of noalloc_scratch_bytes()
// bytes per GPU.  noalloc_scratch() returns its device address on the current device (looked up
// once per device and kept).
// Host-side launch geometry of one level (no device work): every colour-pass workgroup of every
// colour and launch shape maps to patches of that colour inside the grid, covers each patch once
// and stays within the kernels' 32-bit offsets; every operator and transfer launch fits its
// launcher's limits.  False with a reason otherwise; *blocks adds the workgroups enumerated.
bool check_colour_launches(const LevelGeom& g, long long* blocks, std::string* why);
bool check_grid_launches(const LevelGeom& g, std::string* why);
size_t noalloc_scratch_bytes();
hipError_t noalloc_scratch(void** out);
hipError_t launch_zero_boundary(const LevelGeom& g, int prec, void* y, hipStream_t st);
hipError_t launch_rhs_separable(const LevelGeom& g, int prec, int nterms, const double* G, const double* coef, void* b,
                                hipStream_t st);

// Partial sums (nparts doubles) of the squared L2 error, cellwise nq-point Gauss (see grid.hip).
hipError_t launch_l2_error(const LevelGeom& g, const double* x, const double* V, const double* wq, const double* S,
                           const double* uc, int nmodes, int nq, double* partial, int nparts, hipStream_t st);

// vector.hip
int reduction_parts();  // partial slots the reductions use (pairs: 2x this many doubles)
hipError_t launch_fill(int prec, void* x, long long n, double v, hipStream_t st);
hipError_t launch_cast(int from_prec, const void* src, void* dst, long long n, hipStream_t st);
// dst = interior of src, out = |dst|^2, *bad |= non-finite entries; optionally dst32 = (float)dst
// and zero = 0 over the same range; host, host_bad: pinned copies of out[0] and *bad
hipError_t launch_copy_interior_norm(int dim, long long n1d, const double* src, double* dst, double* partial,
                                     double* out, int* bad, hipStream_t st, float* dst32 = nullptr,
                                     double* zero = nullptr, double* host = nullptr, int* host_bad = nullptr);
hipError_t launch_dot2(const double* a, const double* b, const double* c, const double* d, long long n,
                       double* partial, double* out, hipStream_t st, double* host = nullptr);
// The partials of a.b (b FP64, or the FP32 b32 widened exactly, when non-null) only: dot_parts(n) pairs, sum in slot 0.
hipError_t launch_dot_parts(const double* a, const double* b, const float* b32, long long n, double* partial,
                            hipStream_t st);
int dot_parts(long long n);
// x += alpha p, r -= alpha q with alpha = rz / pq (rz: sc[RZNew]; pq: the sum of n_pq entries of pq_part at the
// stride, or sc[PQ] when n_pq is 0), r.r, r.z and pq to sc and rz to sc[RZ], all of what the stopping test reads also to
// host, and r32 = (float) r when r32 != null.  z is the previous preconditioned residual: the FP32 z32 (widened
// exactly) when non-null, else the FP64 z.  pq_part and partial do not overlap.
hipError_t launch_cg_update(double* x, double* r, const double* p, const double* q, const double* z, const float* z32,
                            long long n, const double* pq_part, int n_pq, int pq_stride, double* sc, double* partial,
                            float* r32, double* host, hipStream_t st);
// p = z + beta p (z32 widened exactly when non-null, else z), beta = (rz_new - flexible r.z_old) / rz with rz_new, which
// becomes sc[RZNew], the sum of the partials of r.z; first: p = z.
hipError_t launch_cg_direction(double* p, const double* z, const float* z32, long long n, const double* rz_part,
                               bool flexible, bool first, double* sc, hipStream_t st);

}  // namespace vps
