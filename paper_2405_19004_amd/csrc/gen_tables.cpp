// Build-time generator: prints the 1D patch tables of every degree (computed by tables.cpp) as
// constexpr arrays, so that the colour-pass kernel can use the matrix entries as instruction
// literals instead of loading them from memory.  Run by build.py; the output is a build artifact.
#include <cmath>
#include <cstdio>
#include <cstdlib>

#include "tables.hpp"

namespace {

void emit(const char* type, const char* name, const std::vector<double>& v, const char* fmt) {
  std::printf("  static constexpr %s %s[%zu] = {", type, name, v.size());
  for (size_t i = 0; i < v.size(); ++i) {
    std::printf(i ? ", " : "");
    std::printf(fmt, v[i]);
  }
  std::printf("};\n");
}

}  // namespace

int main() {
  std::printf("// Generated by gen_tables.cpp from tables.cpp; do not edit.\n#pragma once\n\n");
  std::printf("namespace vps {\nnamespace gen {\n\n");
  std::printf("// Patch tables of degree K in precision T: Mc, Ac (interior rows x closure columns); the eigenbasis\n"
              "// (eigen_basis in tables.hpp: the K even eigenvectors first, then the K-1 odd ones) S, lam;\n"
              "// W = S^T M on the interior columns; mu, al = S^T M, S^T A at the left closure end (times +1 / -1\n"
              "// for an even / odd vector at the right end); be = al - lam mu.\n");
  std::printf("template <typename T, int K>\nstruct PatchTables;\n\n");
  for (int k = 1; k <= vps::kMaxDegree; ++k) {
    const vps::Tables1D& t = vps::tables_for_degree(k);
    for (int f = 0; f < 2; ++f) {
      const char* type = f ? "float" : "double";
      const char* fmt = f ? "%.9ef" : "%.17e";
      std::printf("template <>\nstruct PatchTables<%s, %d> {\n", type, k);
      emit(type, "Mc", t.Mc, fmt);
      emit(type, "Ac", t.Ac, fmt);
      const int m = 2 * k - 1, n = 2 * k + 1;
      const vps::EigenBasis e = vps::eigen_basis(k, f == 1);
      std::vector<double> W(m * m), mu(m), al(m), be(m);
      for (int a = 0; a < m; ++a) {
        for (int i = 0; i < m; ++i) W[a * m + i] = e.Mt[a * n + i + 1];
        mu[a] = e.Mt[a * n];
        al[a] = e.At[a * n];
        be[a] = e.be[a];
      }
      emit(type, "S", e.S, fmt);
      emit(type, "W", W, fmt);
      emit(type, "lam", e.lam, fmt);
      emit(type, "mu", mu, fmt);
      emit(type, "al", al, fmt);
      emit(type, "be", be, fmt);
      std::printf("};\n\n");
    }
  }
  std::printf("// Cell tables of degree K in precision T: reference stiffness Ah and mass Mh ((K+1)^2),\n"
              "// prolongation P ((2K+1) x (K+1): phi_a at fine position q of a coarse cell), band rows of the\n"
              "// assembled 1D stiffness / mass (K x (2K+1)) and of the restriction (K x (4K+1)); RA, RM = P^T times\n"
              "// the stiffness / mass of a coarse cell's two fine cells ((K+1) x (2K+1)).\n");
  std::printf("template <typename T, int K>\nstruct CellTables;\n\n");
  for (int k = 1; k <= vps::kMaxDegree; ++k) {
    const vps::Tables1D& t = vps::tables_for_degree(k);
    for (int f = 0; f < 2; ++f) {
      const char* type = f ? "float" : "double";
      const char* fmt = f ? "%.9ef" : "%.17e";
      std::printf("template <>\nstruct CellTables<%s, %d> {\n", type, k);
      emit(type, "Ah", t.Ahat, fmt);
      emit(type, "Mh", t.Mhat, fmt);
      emit(type, "P", t.P, fmt);
      emit(type, "Ab", t.Aband, fmt);
      emit(type, "Mb", t.Mband, fmt);
      emit(type, "Rb", t.Rband, fmt);
      const int np = k + 1, nf = 2 * k + 1;
      for (int which = 0; which < 2; ++which) {
        const std::vector<double>& cell = which ? t.Mhat : t.Ahat;
        std::vector<double> R(np * nf);
        for (int a = 0; a < np; ++a)
          for (int j = 0; j < nf; ++j) {
            long double v = 0;
            for (int c = 0; c < 2; ++c) {
              const int jj = j - c * k;
              if (jj < 0 || jj > k) continue;
              for (int i = 0; i < np; ++i) v += (long double)t.P[(c * k + i) * np + a] * cell[i * np + jj];
            }
            R[a * nf + j] = (double)v;
          }
        emit(type, which ? "RM" : "RA", R, fmt);
      }
      std::printf("};\n\n");
    }
  }
  std::printf("}  // namespace gen\n}  // namespace vps\n");
  return 0;
}
