// Host setup of the algebraic multigrid preconditioner for the scalar-potential
// solve: smoothed aggregation (Jacobi-smoothed prolongation on the first
// `smooth_levels` levels, plain aggregation below), Galerkin coarse
// operators, dense inverse on the coarsest level.
#pragma once
#include <algorithm>
#include <atomic>
#include <cstdint>
#include <functional>
#include <vector>

namespace mmsd {

struct Csr {
  int nrows = 0, ncols = 0;
  std::vector<int> rp, ci;
  std::vector<double> v;
};

struct AmgLevel {
  Csr A;                   // operator of this level
  std::vector<double> dinv;
  double omega = 0;        // prolongation smoothing weight 4 / (3 rho(D^-1 A))
  double wsmooth = 0;      // the V-cycle smoother's damped-Jacobi weight (amg_setup)
  Csr P;                   // prolongation to this level from the next coarser one
  Csr R;                   // restriction, the transpose of P
  Csr AP;                  // A P (formed for the Galerkin product; post-smoothing sweeps it)
};

struct AmgHierarchy {
  std::vector<AmgLevel> lv;      // levels 0 .. L-1 (each with P/R to level l+1)
  int nc = 0;                    // size of the coarsest level L
  std::vector<double> Ainv;      // dense inverse of the coarsest operator, row-major
  double complexity = 0;         // total nonzeros of all operators / nonzeros of A_0
};

struct AmgParams {
  double theta = 0.04;           // strength of connection |a_ij| >= theta sqrt(a_ii a_jj)
  int smooth_levels = 10;        // levels whose prolongation is Jacobi-smoothed (all, with p_drop)
  int coarse_max = 600;          // stop coarsening at or below this size
  int max_levels = 10;
  double p_drop = 0.1;           // drop smoothed-P entries below this fraction of the row's largest
  // The V-cycle smoother's weight: smooth_scale x omega, capped at 1.9 / g
  // with g a Gershgorin bound of rho(D^-1 A) (the smaller of those of D^-1 A
  // and of D^-1/2 A D^-1/2), so that the damped Jacobi sweep stays
  // convergent whatever the power iteration's estimate of rho.  In a CPU
  // model of the preconditioned CG (to 1e-10 from zero), 1.2 x omega took 24
  // instead of 26 iterations on the 80 nm cube and 27 instead of 28 on the
  // polycrystal (where the cap binds on the two coarsest levels); 1.3 x was
  // no better and 1.45 x diverged.
  double smooth_scale = 1.2;
};

// Runs f(a, b) over [0, n) cut into contiguous ranges, on up to 16 threads
// (one for n < 2048), and on the calling thread's share of the cores when a
// sharing counter is set (below).  A thread that cannot be started leaves its
// range and the rest to the calling one.  With a grain, on at most one thread per
// `grain` items, however few those are: starting a thread costs as much as
// some ten thousands of entries of a light loop (matrix rows looked at, copied or
// sorted).  light_rows is the grain of such a loop over the rows of a matrix
// with `entries` entries: by entries, since rows hold 7 (a Kuhn mesh's potential
// matrix) to 50 of them (the fused post-smoothing of a Delaunay mesh, whose
// slices were filled in 5.7 ms with a grain of 8,192 rows and 64-bit zeros
// written first, and are in 2.9 ms).  kLight: the grain of loops over row lengths
// alone.
constexpr int64_t kLight = 8192, kLightEntries = 65536;
inline int64_t light_rows(int64_t rows, int64_t entries) {
  return std::max<int64_t>(1, rows * kLightEntries / std::max<int64_t>(1, entries));
}
void parallel_for(int64_t n, const std::function<void(int64_t, int64_t)>& f, int64_t grain = 0);

// Threads that share the cores: while `active` is set on a thread, its
// parallel_for calls use at most cores / *active threads (the server's setup
// workers set it to their count of busy workers).  nullptr: no sharing.
void share_cores(const std::atomic<int>* active);

// A coupling a_ij is as good as zero when |a_ij| <= kZeroCoupling min(a_ii, a_jj):
// below the rounding error of its own assembled sum, whose terms are of the
// diagonal's size.
constexpr double kZeroCoupling = 0x1p-52;

// The matrix (rp, ci, v) without the couplings that are as good as zero; its
// diagonal in diag.  On a box cut into Kuhn tetrahedra the face and space
// diagonals carry no coupling (the P1 gradients of their end points are
// orthogonal, also under the shell's diagonal metric): 6.9 of the 14.6
// entries per row of the 80 nm cube's potential matrix remain, the others are
// exact zeros.  The device sweeps and the multigrid setup read the rest
// only.  Entries keep their order, so with exact zeros every sum has the
// same bits as before.  The rows of A P shrink from 14.3 to 9.0 entries and
// those of the next operator from 37.7 to 25.6 with them.  Measured: 14
// evaluations of the polycrystal 245.1 -> 193.6 ms, four field points of the
// 80 nm cube 94.0 -> 81.3 ms.
Csr without_zero_couplings(const std::vector<int>& rp, const std::vector<int>& ci, const std::vector<double>& v,
                           std::vector<double>* diag);

// T = (I - W A) P, W = wsmooth D^-1: what the post-smoothing adds per coarse
// value, x = W b + W (b - A W b) + T x_{l+1}.  Rows with ascending columns, the
// union of the patterns of A P and P.
Csr smoothed_prolongation(const AmgLevel& L);

// M = R (I - A W), W = wsmooth D^-1: the restriction of the residual left by
// one damped-Jacobi sweep from zero, b_{l+1} = M b_l.  For symmetric A it is
// the transpose of T = (I - W A) P (given, or formed); rows with ascending
// columns.
Csr residual_restriction(const AmgLevel& L, const Csr* T = nullptr);

// [2 I - W A | T] (T the smoothed_prolongation): the pre-smoothing, its
// residual and the post-smoothing in one matrix over [W b | x_{l+1}], since
// W b + W (b - A W b) = 2 W b - W A (W b).  Columns of T are shifted by n.
Csr fused_post_smoothing(const AmgLevel& L, const Csr& T);

// Build the hierarchy for the symmetric positive definite CSR matrix A
// (taken by value: pass a moved copy to spare one).  Returns false (and
// leaves h empty) when the matrix does not coarsen.
bool amg_setup(Csr A, const AmgParams& prm, AmgHierarchy* h);

}  // namespace mmsd
