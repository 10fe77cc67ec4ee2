// Host check of the matrices the device's V(1,1) cycle sweeps, on the
// hierarchy of a CSR matrix (int32 n, int32 nnz, rp, ci, values in argv[1]):
// per level, for seeded b and x and W = wsmooth D^-1, the largest relative
// deviation of
//   post   W (b + res) + T x from xa + W (b - A xa), xa = W b + P x,
//          res = b - A W b, T = smoothed_prolongation
//   fused  [2 I - W A | T] [W b | x] (fused_post_smoothing) from the same
//   adj    y . T x from (M y) . x, M = residual_restriction
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

static double rel(const std::vector<double>& a, const std::vector<double>& b) {
  double d = 0, m = 0;
  for (size_t i = 0; i < a.size(); ++i) {
    d = std::fmax(d, std::fabs(a[i] - b[i]));
    m = std::fmax(m, std::fabs(a[i]));
  }
  return m > 0 ? d / m : d;
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
  std::mt19937_64 g(5);
  std::normal_distribution<double> N01;
  for (size_t l = 0; l < h.lv.size(); ++l) {
    const AmgLevel& L = h.lv[l];
    const int nl = L.A.nrows, nn = L.P.ncols;
    std::vector<double> b(nl), x(nn), wb(nl), res(nl), xa(nl), z(nl), zt(nl);
    for (auto& e : b) e = N01(g);
    for (auto& e : x) e = N01(g);
    for (int i = 0; i < nl; ++i) wb[i] = L.wsmooth * L.dinv[i] * b[i];
    const std::vector<double> Awb = spmv(L.A, wb), Px = spmv(L.P, x);
    for (int i = 0; i < nl; ++i) {
      res[i] = b[i] - Awb[i];
      xa[i] = wb[i] + Px[i];
    }
    const std::vector<double> Axa = spmv(L.A, xa);
    const Csr T = smoothed_prolongation(L);
    const std::vector<double> Tx = spmv(T, x);
    double yt = 0, my = 0, sc = 0;
    for (int i = 0; i < nl; ++i) {
      const double w = L.wsmooth * L.dinv[i];
      z[i] = xa[i] + w * (b[i] - Axa[i]);
      zt[i] = w * (b[i] + res[i]) + Tx[i];
      yt += b[i] * Tx[i];
      sc += std::fabs(b[i] * Tx[i]);
    }
    std::vector<double> y(wb);
    y.insert(y.end(), x.begin(), x.end());
    const Csr C = fused_post_smoothing(L, T);
    const std::vector<double> zc = spmv(C, y), Mb = spmv(residual_restriction(L), b);
    for (int i = 0; i < nn; ++i) my += Mb[i] * x[i];
    std::printf("level %zu rows %d post %.3e fused %.3e adj %.3e\n", l, nl, rel(z, zt), rel(z, zc),
                std::fabs(yt - my) / sc);
  }
  return 0;
}
