// Host-only rules of the DACP path: parameter selection, the acceptance rule and the
// bookkeeping of the divide-and-conquer merge.  No HIP types: this part is compiled with the
// host compiler, both into the library and into the sanitizer harness of the test suite.
#pragma once

#include <cstdint>
#include <functional>
#include <vector>

#include "../../include/dacp.h"

namespace dacp {
namespace rules {

// Estimated number of levels in [-a_r E_b, a_r E_b] from Jackson-damped Chebyshev moments of the
// density (kernel polynomial method; closed-form integral of every term).
double kpm_count(const std::vector<double> &mu, int64_t D, double a_r);
// Smallest a_r in (0, 1) whose estimated count reaches `count` (bisection).
double window_for_count(const std::vector<double> &mu, int64_t D, double count);
// Sampled evolution orders k_j = 2 floor(j pi / (2 a_r)), j = 1..n (App. B, App. C: even orders).
std::vector<int64_t> sample_orders(double a_r, int n);

// Window, filter order and basis size of one attempt (Sec. II.A, II.B, III).
struct Plan {
  double n_w, a_r, a;
  int K, b, n, m;
};
Plan make_plan(const dacp_opts &o, int64_t D, int N, double e_b, const std::vector<double> &mu, double window_ratio,
               int attempt);

// Positions of theta sorted by (|theta|, theta).
std::vector<int> central_order(const std::vector<double> &theta);

// Result of the acceptance rule (accept_rule).
struct AcceptResult {
  std::vector<char> ok, ghost;  // per Ritz value (index into theta)
  std::vector<double> est;      // per candidate position q < n_sel (INFINITY for a ghost)
  std::vector<int> core_idx;    // candidate positions of the contiguous core, walking outward
  double max_est = 0.0;
  int n_ghost = 0;
};

// Largest number of neighbouring Ritz values grouped into one cluster by accept_rule.
constexpr int kAcceptMaxCluster = 8;

// The acceptance rule (Sec. II.C residual check with a quadratic residual bound).
//   theta[r]      Ritz values, ascending
//   order         central_order(theta)
//   rnorm[n_sel]  residual norms ||H phi - theta phi|| of the unit Ritz vectors of the first n_sel
//                 positions of `order` (the candidates)
//   a, tol        window half-width and accepted error
// Rule:
//   * A candidate is a ghost when rnorm >= a - |theta|: a unit vector made only of eigenvectors
//     outside the window [-a, a] has exactly that residual or more, so such a Ritz value may
//     approximate no level at all.  Below it, Weyl's bound puts a level of H within rnorm of theta,
//     inside the window.
//   * Estimate (block quadratic residual bound): for a cluster C of consecutive non-ghost Ritz
//     values with orthonormal Ritz vectors X_C and residual block R_C, the |C| eigenvalues of H
//     paired with them lie within ||R_C||^2 / delta_C, delta_C being the distance from C to the rest
//     of the spectrum.  Here ||R_C||^2 <= sum of rnorm^2 over C, and the rest of the spectrum is
//     represented by the non-ghost Ritz values outside C (each moved towards C by its own residual,
//     zero where it is not a candidate) and by the window edges (levels beyond +-a are not
//     resolved).  The estimate of a candidate is the smallest of rnorm and this bound over every
//     run C of at most kAcceptMaxCluster candidates that contains it.  Accepted: estimate <= tol.
//   * Core: walk the candidates outward in |theta| while |theta| <= a; the first candidate that is
//     a ghost or not accepted ends it.
AcceptResult accept_rule(const std::vector<double> &theta, const std::vector<int> &order, int n_sel,
                         const std::vector<double> &rnorm, double a, double tol);

// Number of runs of at least b consecutive values of the ascending list eigs[n] in which each
// value lies within 2 tol of the next (levels of multiplicity b at the accepted accuracy).
int clusters_at_width(const double *eigs, int n, double tol, int b);

// Divide-and-conquer merge bookkeeping (host side of the rank-one update): sort the two halves'
// eigenvalues, deflate tiny z components and close pairs (Givens rotations that zero one z of
// the pair), and list the non-deflated problem.
//   dv[n]       eigenvalues of the two solved halves in block order
//   z[n]        the update vector, normalised; rho > 0 the update weight
//   lo          absolute row of the block's first eigenvector
// Outputs: sorted values ds/zs with their absolute rows rowid; defl[j] = 1 for a deflated
// sorted entry; rotations as row pairs (rot_pq) and (c, s) (rot_cs), applied in order; nd = the
// sorted positions that stay in the secular problem.
struct DcDeflation {
  std::vector<double> ds, zs;
  std::vector<int> rowid;
  std::vector<char> defl;
  std::vector<int> rot_pq;
  std::vector<double> rot_cs;
  std::vector<int> nd;
};
DcDeflation dc_deflate(const std::vector<double> &dv, const std::vector<double> &z, double rho, int lo);

// Final placement after a merge: entries (value, kind, index) with kind 0 = deflated (index = an
// absolute row) and kind 1 = secular root (index = position in the non-deflated list), sorted by
// value (stable).  Gives, per output row t of the block, where it comes from.
struct DcEntry {
  double v;
  int kind, idx;
};
struct DcPlacement {
  std::vector<int> src_defl, dst_defl;  // deflated: source absolute row -> block row
  std::vector<int> dst_of_root;         // root q -> block row
  std::vector<double> w;                // eigenvalue of block row t
};
DcPlacement dc_place(std::vector<DcEntry> ents, int k);

// Moment projection from a stored basis (App. C, Eq. shift): with T_A T_x = (T_{A+x} + T_{|A-x|}) / 2,
// the Gram block of an anchor panel of order A with a stored panel of order x gives the moment at
// one of A + x, |A - x| once the moment at the other is known (both at once when A or x is 0).
// Anchor orders for the uniform grid whose last sample is kn: 0, 1, 2, kn - 2 .. kn + 1, ascending
// and distinct.
std::vector<int64_t> anchor_orders(int64_t kn);
// The derivation chain for panel orders `orders` (orders[0] = 0, last = kn): sweeping the (anchor,
// panel) pairs until nothing new follows, each moment is derived once, from the first pair that
// reaches it; only the rules that the orders x + y, |x - y| of two panel orders need (and those
// they are derived from) are kept, in the order found, so a rule's other moment comes before it.
struct MomentChain {
  std::vector<int> table;           // per kept rule: anchor index, panel index, earlier rule or -1
  std::vector<int64_t> order;       // per kept rule: the order of the moment it gives
  std::vector<int> block_of;        // order k = 0 .. 2 kn: the kept rule giving moment k, or -1
  int64_t missing = -1;             // an order the assembly needs that the anchors do not reach
};
MomentChain moment_chain(const std::vector<int64_t> &orders, const std::vector<int64_t> &anchors);

// Column groups of a recurrence over b columns of D rows, `g` wanted per group.  The fused kernels take
// power-of-two widths (fused(w)), so a ragged width is rounded up to w and the columns past b are zero
// (they cost no launch, where the general kernels take twice as long per step), and `per` groups advance
// in one launch.  One group of 8 columns is 2 to 32 MB a block below 2^19 rows, whose launches are bound by
// their own start and end (6-8 us each at 2^16 rows, the streams' rate would take 2.5); together they
// stream at the rate of a large copy.  A launch's groups stay within the 256 MB Infinity Cache (col_bytes
// a row and column over the live blocks): past it every step would go to HBM (two groups at once at 2^20
// rows: 50-60 us a group, alone 43); half of it costs the FP64 filter at 2^17 to 2^19 rows 5-8 %.
//
// The columns left over by whole groups go along with them as one more padded group, or, where that moves
// more than a launch costs, in a launch of their own of the next power of two (tail columns of width
// tail_w; without a fused plan for it the general kernels at their own number).  A launch of their own is
// always right when the padded group would need one too; else from kPadRows padded rows on: 9 columns of 2^20
// rows took 10.8 ms padded to 16 and 8.4 as 8 and 1; 9 of 2^17 rows 1.7 and 2.2 (evolution); the filter's
// four launches an order put the line higher (9 of 2^18: 6.4 and 7.2), and in mixed precision, where widths
// below 4 have no fused plan, sharing a launch is right at any size (9 of 2^19: 10.0 and 12.3).
// Mixed precision: a padded group alone of less than 4 MB in FP32 is slower than the general kernels at the
// ragged width (5 columns of 2^16 rows: 2.2 against 1.9 ms).
constexpr int64_t kRecCacheBytes = int64_t(256) << 20;
constexpr int64_t kPadRows = int64_t(5) << 18, kPadRowsFilter = int64_t(2) << 20;
struct ColumnPlan {
  int g, per;
  bool fused;
  int tail, tail_w;
};
ColumnPlan column_plan(int64_t D, int b, int g, int64_t col_bytes, bool mixed, bool filter,
                       const std::function<bool(int)> &fused);

// Route of a recurrence up to 14 spins: a workgroup per column on chip (batch.hip), or the kernels that
// step through memory, spread over the GPU.  Microseconds of one apply, fitted to what both took on
// MI355X for 8 to 14 spins and 1 to 256 columns of a chain (single-spin flips), the paper's
// nearest-neighbour model (L - 1 pair flips) and its spin glass (L (L - 1) / 2), and both with X_i X_j +
// Y_i Y_j (twice as many flips, half of them with a sign):
//   on chip  0.45 + rows / 2^14 (1.9 + 3.3 with single-spin flips + 0.49 a flip of the table, 0.84 with a
//            sign), for every compute unit's worth of columns: a table flip is a sweep of the column through
//            one unit's LDS (at 14 spins 5.7; 8.8 and 46.7; 20 and 124);
//   memory   launches of 5.8 and 0.22 a flip with a sign, or 0.23 a flip where those are many, and the
//            reads of each flip mask and 12 streams at 16 TB/s of the caches, half hidden under one
//            another (the 2/3 power of their 3/2 powers' sum; for one column 6.0; 6.3 and 21; 8.9 and
//            40; for 64 13; 13 and 51; 18.5 and 92).
struct FlipCounts {
  int flips = 0, masks = 0;              // all, and their distinct x-masks
  int table_plain = 0, table_signed = 0;  // those that are not a single spin's without a sign
};
double onchip_apply_us(int L, const FlipCounts &f);
double memory_apply_us(int L, const FlipCounts &f, int b);
// Whether `applies` applies to each of b columns are faster on chip; extra_us: what the other route spends
// besides an apply (scalars kept between launches).  Never past kOnChipSeconds in one launch, which
// holds its compute units until it ends.
constexpr double kOnChipSeconds = 2.0;
bool onchip_pays(int L, const FlipCounts &f, int b, int cus, double applies, double extra_us);

}  // namespace rules
}  // namespace dacp
