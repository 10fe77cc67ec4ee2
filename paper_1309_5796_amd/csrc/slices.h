// Slices: the layout in which the device holds the matrices of the potential
// solve (host side).
#pragma once
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <memory>
#include <vector>

#include "amg.h"

namespace mmsd {

// A CSR matrix in slices of one wavefront, W lanes per row (1: 64 rows per
// slice): slice s starts at so[s] and is as wide as its longest row; entry k
// of its row r is at so[s] + 64 (k / W) + r W + k mod W; the rest is padded
// with the row's own column (clamped to the column range) and a zero value.
// Slices are built in parallel, and each value is written once: the arrays
// start without one, so that their pages are first touched by those threads.
template <typename T>
struct Unset : std::allocator<T> {
  template <typename U>
  struct rebind {
    using other = Unset<U>;
  };
  template <typename U>
  void construct(U*) noexcept {}
};
struct Sliced {
  std::vector<int> so;
  std::vector<int, Unset<int>> sc;
  std::vector<double, Unset<double>> sv;
  std::vector<int> order;   // row at each position (empty: position = row)
};

// Rows sorted by length, longest first, inside windows of kOrderWindow rows:
// a slice is as wide as its longest row, and the multigrid's matrices mix row
// lengths (aggregates of 5-47 fine nodes, rows of A P next to aggregate
// boundaries), so that sorting cuts the padding.  But neighbouring lanes then
// hold rows further apart, whose gathers and own values share fewer cache
// lines: with windows of 512 rows the polycrystal's post-smoothing of the
// finest level took 84 us, with 256 82.6 us, with 128 76.8 us, within a slice
// 77.7 us, its 14 evaluations 157.4, 155.1, 152.2 and 153.1 ms.
constexpr int kOrderWindow = 128;
inline std::vector<int> window_order(const std::vector<int>& len) {
  const int64_t n = (int64_t)len.size();
  std::vector<int> order(n);
  for (int64_t i = 0; i < n; ++i) order[i] = (int)i;
  parallel_for((n + kOrderWindow - 1) / kOrderWindow, [&](int64_t a, int64_t b) {
    for (int64_t w = a; w < b; ++w) {
      auto first = order.begin() + w * kOrderWindow;
      auto last = order.begin() + std::min<int64_t>(n, (w + 1) * kOrderWindow);
      std::stable_sort(first, last, [&](int x, int y) { return len[x] > len[y]; });
    }
  }, kLight / kOrderWindow);
  return order;
}
// Offsets of the slices of a CSR pattern (W lanes per row), 32-bit as the
// sweeps index them; none when they need more (the potential matrix has the
// same limit).
inline std::vector<int> slice_offsets(const std::vector<int>& rp, int W = 1) {
  const int64_t n = (int64_t)rp.size() - 1, rows = 64 / W, ns = (n + rows - 1) / rows;
  std::vector<int> so(ns + 1, 0);
  parallel_for(ns, [&](int64_t a, int64_t b) {
    for (int64_t sl = a; sl < b; ++sl) {
      int w = 0;
      for (int64_t i = rows * sl; i < std::min<int64_t>(n, rows * (sl + 1)); ++i) w = std::max(w, rp[i + 1] - rp[i]);
      so[sl + 1] = (w + W - 1) / W;
    }
  }, light_rows(ns, rp[n]));
  int64_t total = 0;
  for (int64_t sl = 1; sl <= ns; ++sl) {
    total += 64LL * so[sl];
    if (total > INT32_MAX) return {};
    so[sl] = (int)total;
  }
  return so;
}

inline Sliced make_sliced(const std::vector<int>& rp, const std::vector<int>& ci, const std::vector<double>& v,
                   int ncols, int W = 1, bool ordered = false) {
  const int64_t n = (int64_t)rp.size() - 1, rows = 64 / W, ns = (n + rows - 1) / rows;
  const int lw = std::ilogb(W);   // W is a power of two
  Sliced S;
  if (ordered) {
    std::vector<int> len(n);
    for (int64_t i = 0; i < n; ++i) len[i] = rp[i + 1] - rp[i];
    S.order = window_order(len);
    std::vector<int> rpo(n + 1, 0);   // row starts of the rows in position order (lengths only matter)
    for (int64_t q = 0; q < n; ++q) rpo[q + 1] = rpo[q] + len[S.order[q]];
    S.so = slice_offsets(rpo, W);
  } else {
    S.so = slice_offsets(rp, W);
  }
  if (S.so.empty()) return S;   // too large
  S.sc.resize(S.so[ns]);
  S.sv.resize(S.so[ns]);
  parallel_for(ns, [&](int64_t a, int64_t b) {
    for (int64_t sl = a; sl < b; ++sl) {
      const int w = (S.so[sl + 1] - S.so[sl]) / 64;
      for (int r = 0; r < rows; ++r) {
        const int64_t pos = rows * sl + r;
        const int64_t i = pos < n && ordered ? S.order[pos] : pos;
        const int len = pos < n ? rp[i + 1] - rp[i] : 0;
        for (int k = 0; k < w * W; ++k) {
          const int64_t q = S.so[sl] + 64LL * (k >> lw) + r * W + (k & (W - 1));
          if (k < len) {
            S.sc[q] = ci[rp[i] + k];
            S.sv[q] = v[rp[i] + k];
          } else {
            S.sc[q] = (int)std::min<int64_t>(i, ncols - 1);
            S.sv[q] = 0.0;
          }
        }
      }
    }
  }, light_rows(ns, rp[n]));
  return S;
}

}  // namespace mmsd
