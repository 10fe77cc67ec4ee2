// Host check of the restriction M that a fused level's DOWN sweeps, on the
// hierarchy of a CSR matrix (int32 n, int32 nnz, rp, ci, values in argv[1]) as
// problem creation builds it: per level, for a seeded b, the largest relative
// deviation of M b from R (b - A W b), with the residual formed by A itself.
#include <cmath>
#include <cstdio>
#include <random>
#include <vector>

#include "amg.h"

using namespace mmsd;

static std::vector<double> spmv(const Csr& A, const std::vector<double>& x) {
  std::vector<double> y(A.nrows, 0.0);
  for (int i = 0; i < A.nrows; ++i)
    for (int k = A.rp[i]; k < A.rp[i + 1]; ++k) y[i] += A.v[k] * x[A.ci[k]];
  return y;
}

int main(int argc, char** argv) {
  if (argc < 2) return 2;
  FILE* f = std::fopen(argv[1], "rb");
  if (!f) return 2;
  int n = 0, nnz = 0;
  std::vector<int> rp, ci;
  std::vector<double> v, diag;
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
  AmgHierarchy h;
  if (!amg_setup(without_zero_couplings(rp, ci, v, &diag), AmgParams{}, &h)) return 3;
  std::mt19937_64 g(7);
  std::normal_distribution<double> N01;
  for (const AmgLevel& L : h.lv) {
    const int nl = L.A.nrows;
    std::vector<double> b(nl), w(nl), res(nl);
    for (int i = 0; i < nl; ++i) {
      b[i] = N01(g);
      w[i] = L.wsmooth * L.dinv[i] * b[i];
    }
    const std::vector<double> Aw = spmv(L.A, w);
    for (int i = 0; i < nl; ++i) res[i] = b[i] - Aw[i];
    const Csr T = smoothed_prolongation(L);
    const std::vector<double> want = spmv(L.R, res), got = spmv(residual_restriction(L, &T), b);
    double dev = 0, top = 0;
    for (size_t i = 0; i < want.size(); ++i) {
      dev = std::fmax(dev, std::fabs(got[i] - want[i]));
      top = std::fmax(top, std::fabs(want[i]));
    }
    std::printf("rows %d dev %.3e\n", nl, dev / top);
  }
  return 0;
}
