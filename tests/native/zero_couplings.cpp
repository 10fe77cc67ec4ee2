// Host check of without_zero_couplings.  Reads a CSR matrix (int32 n, int32
// nnz, rp, ci, values) from argv[1] and prints the kept entries, whether the
// kept pattern is symmetric with every diagonal in it, the diagonal's
// largest deviation, the largest |dropped| / min(a_ii, a_jj), and whether the
// product with a seeded vector has the same bits.
#include <cmath>
#include <cstdio>
#include <random>
#include <vector>

#include "amg.h"

using namespace mmsd;

int main(int argc, char** argv) {
  if (argc < 2) return 2;
  FILE* f = std::fopen(argv[1], "rb");
  if (!f) return 2;
  int n = 0, nnz = 0;
  std::vector<int> rp, ci;
  std::vector<double> v;
  bool ok = std::fread(&n, 4, 1, f) == 1 && std::fread(&nnz, 4, 1, f) == 1;
  if (ok) {
    rp.resize(n + 1);
    ci.resize(nnz);
    v.resize(nnz);
    ok = std::fread(rp.data(), 4, n + 1, f) == (size_t)n + 1 && std::fread(ci.data(), 4, nnz, f) == (size_t)nnz &&
         std::fread(v.data(), 8, nnz, f) == (size_t)nnz;
  }
  std::fclose(f);
  if (!ok) return 2;
  std::vector<double> d;
  const Csr Z = without_zero_couplings(rp, ci, v, &d);
  auto has = [&](int i, int j) {
    for (int k = Z.rp[i]; k < Z.rp[i + 1]; ++k)
      if (Z.ci[k] == j) return true;
    return false;
  };
  bool sym = true;
  double ddev = 0, dropped = 0;
  std::mt19937_64 g(11);
  std::normal_distribution<double> N01;
  std::vector<double> x(n);
  for (auto& e : x) e = N01(g);
  bool same = true;
  for (int i = 0; i < n; ++i) {
    double a = 0, b = 0;
    for (int k = rp[i]; k < rp[i + 1]; ++k) {
      a += v[k] * x[ci[k]];
      if (ci[k] == i) ddev = std::fmax(ddev, std::fabs(d[i] - v[k]));
      if (!has(i, ci[k])) dropped = std::fmax(dropped, std::fabs(v[k]) / std::fmin(d[i], d[ci[k]]));
    }
    for (int k = Z.rp[i]; k < Z.rp[i + 1]; ++k) {
      b += Z.v[k] * x[Z.ci[k]];
      sym = sym && has(Z.ci[k], i);
    }
    same = same && a == b && has(i, i);
  }
  std::printf("n %d nnz %d kept %d sym %d ddev %.3e dropped %.3e same %d\n", n, nnz, (int)Z.ci.size(), sym, ddev,
              dropped, same);
  return 0;
}
