// Divide-and-conquer eigen-decomposition of symmetric tridiagonal matrices (Cuppen's tear,
// deflation and the secular equation; eigenvectors of each rank-one update from the Gu-Eisenstat
// recomputed z so they stay orthogonal to working precision), for any number of matrices at once.
//
// What bounds it: a merge of a few hundred rows is microseconds of arithmetic, so the tree is walked
// one depth at a time with every merge of that depth, of every matrix, in the same launches.  A
// depth costs one copy to the host (the update vectors and eigenvalues), the O(n) deflation
// bookkeeping there, one copy back and seven launches; the leaves are solved on the GPU.
// Measured on one matrix of n = 1237 (and its 866-row H~): the merges took 75 ms as one host-driven
// merge after another with a thread per secular root.
//
// Eigenvectors are kept as rows: row lo + j of a block [lo, hi) holds component lo + i at column
// lo + i.  A node of depth t writes buffer t mod 2 (the root, depth 0, the caller's Z), so its
// children, all at depth t + 1, sit in the other one.  Entries outside a node's own columns are
// never read: each merge knows which half every row is supported on.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <numeric>
#include <vector>

#include "host_rules.h"
#include "internal.h"
#include "secular.h"
#include "wave.h"

namespace dacp {

namespace {

constexpr int kLeaf = 32;
constexpr int kDcThreads = 256;  // four waves, one secular root (or row) each

typedef double v4d __attribute__((ext_vector_type(4)));
typedef double v2d __attribute__((ext_vector_type(2)));

// One leaf: rows [lo, hi) of the matrix with diagonal d and off-diagonal e, Z its eigenvector buffer.
struct DcLeaf {
  const double *d, *e;
  double *Z, *w;
  int n, lo, hi;
};

// One rank-one merge of the halves [lo, m) and [m, hi).
struct DcMerge {
  double *Zin, *Zout;  // children's rows, result rows (ld n each)
  double *U, *G;       // eigenvectors of the update and the gathered children's rows (ld n each)
  double *w;           // the matrix's eigenvalues, block row t at w[lo + t]
  double rho;
  int n, lo, m, hi;
  int off;             // offset of this merge in the depth's packed per-row arrays
  int k;               // size of the secular problem
  int k1, k12;         // its rows supported on the first half only / on both (the rest: second half)
  int nrot, rot;       // deflating rotations and their offset
};

// Rotation of rows p and q (absolute); bit 0 / 1 of pf, qf: the row is supported on the first /
// second half when the rotation reads it.
struct DcRot {
  double c, s;
  int p, q, pf, qf;
};

// Packed per-row device arrays of one depth (one slot per block row of every merge).
struct DcRows {
  const double *pole, *z;  // secular problem, ascending poles (k entries)
  const double *dval;      // deflated eigenvalues ascending (n - k entries)
  const int *ucol;         // column of U / row of G of pole i
  const int *src;          // G row q: absolute source row
  const int *dsrc;         // deflated entry t: absolute source row
  const int *dflag;        // deflated entry t: halves its row is supported on (bits 0, 1)
  int *org;
  double *tau, *zh;
  int *rank;               // root j: block row of its eigenvector
};

struct WaveLanes {
  __device__ __forceinline__ int first() const { return threadIdx.x & 63; }
  __device__ __forceinline__ int stride() const { return 64; }
  __device__ __forceinline__ double sum(double v) const { return wave_sum(v); }
};

// Leaf eigenproblem, one wave each: implicit QR with a Wilkinson shift on the torn diagonal, then the
// eigenvalues sorted by counting.  Lane i holds d_i, e_i and component i of every eigenvector (those in
// LDS, row by row); lanes 32.. repeat lanes 0.. .  The chase is one dependent chain, so it reads
// and writes d and e by uniform lane index, with no LDS on it, and one reciprocal square root a
// rotation; where blocks end is read off a ballot.  (d and e in LDS: 330 us for leaves of 20 rows.)
// bad is set when the iteration does not end.
__global__ __launch_bounds__(64) void k_dc_leaf(const DcLeaf *leaves, int *bad) {
  __shared__ double Zs[kLeaf + 1][kLeaf + 1];
  const DcLeaf L = leaves[blockIdx.x];
  const int n = L.hi - L.lo, lane = threadIdx.x;
  const int col = lane & (kLeaf - 1);
  double d = 0.0, e = 0.0;
  if (col < n) {
    d = L.d[L.lo + col];
    // the tears at the block's two ends (|e| taken off both neighbours)
    if (col == 0 && L.lo > 0) d -= fabs(L.e[L.lo - 1]);
    if (col == n - 1 && L.hi < L.n) d -= fabs(L.e[L.hi - 1]);
    if (col + 1 < n) e = L.e[L.lo + col];
  }
  for (int i = 0; i < n; ++i) Zs[i][col] = (i == col) ? 1.0 : 0.0;
  const double eps = 2.220446049250313e-16;
  bool ok = false;
  for (int it = 0; it <= 40 * n + 100; ++it) {
    const double dn = __shfl(d, (col + 1) & (kLeaf - 1), 64);
    const bool coupled = col + 1 < n && !(fabs(e) <= eps * (fabs(d) + fabs(dn)));
    if (!coupled) e = 0.0;
    const uint32_t m = static_cast<uint32_t>(__ballot(coupled));
    if (m == 0) {
      ok = true;
      break;
    }
    // the last unreduced block [p, q]
    const int q = 32 - __clz(static_cast<int>(m));
    const uint32_t below = ~m & ((1u << (q - 1)) - 1u);
    const int p = below ? 32 - __clz(static_cast<int>(below)) : 0;
    const double a = read_lane(d, q - 1), bb = read_lane(e, q - 1), cc = read_lane(d, q);
    const double delta = 0.5 * (a - cc);
    const double den = delta + (delta >= 0.0 ? 1.0 : -1.0) * hypot(delta, bb);
    const double mu = (den != 0.0) ? cc - bb * bb / den : cc;
    double dk = read_lane(d, p), ek = read_lane(e, p);
    double x = dk - mu, z = ek;
    double carry = Zs[p][col], next = Zs[p + 1][col];
    for (int k = p; k < q; ++k) {
      const double dk1 = read_lane(d, k + 1), en = read_lane(e, k + 1);
      const double zn = next;
      next = Zs[k + 2 <= q ? k + 2 : q][col];
      // c x - s z = r, s x + c z = 0
      double c = 1.0, s = 0.0;
      const double big = fmax(fabs(x), fabs(z));
      if (z != 0.0) {
        if (big > 1e-140 && big < 1e140) {
          const double r = rsqrt(x * x + z * z);
          c = x * r;
          s = -z * r;
        } else {
          const double xs = x / big, zs = z / big, r = rsqrt(xs * xs + zs * zs);
          c = xs * r;
          s = -zs * r;
        }
      }
      if (k > p && col == k - 1) e = c * x - s * z;
      const double dnew = c * c * dk - 2.0 * c * s * ek + s * s * dk1;
      const double off = c * s * (dk - dk1) + (c * c - s * s) * ek;
      dk = s * s * dk + 2.0 * c * s * ek + c * c * dk1;
      if (col == k) {
        d = dnew;
        e = off;
      }
      if (k < q - 1) {
        x = off;
        z = -s * en;
        ek = c * en;
      }
      Zs[k][col] = c * carry - s * zn;
      carry = s * carry + c * zn;
    }
    if (col == q) d = dk;
    Zs[q][col] = carry;
  }
  if (!ok && lane == 0) *bad = 1;
  __syncthreads();
  for (int r = 0; r < n; ++r) {
    const double v = read_lane(d, r);
    const uint32_t before = static_cast<uint32_t>(__ballot(col < n && (d < v || (d == v && col < r))));
    const int rank = __popc(before);
    if (lane == 0) L.w[L.lo + rank] = v;
    if (lane < n) L.Z[static_cast<int64_t>(L.lo + rank) * L.n + L.lo + lane] = Zs[r][lane];
  }
}

// z = [last component of the first half's rows; first component of the second half's].
__global__ void k_dc_z(const DcMerge *merges, double *z) {
  const DcMerge M = merges[blockIdx.y];
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= M.hi - M.lo) return;
  const int c = (M.lo + i < M.m) ? M.m - 1 : M.m;
  z[M.off + i] = M.Zin[static_cast<int64_t>(M.lo + i) * M.n + c];
}

// The deflating rotations in order, one column per thread: row_p <- c row_p - s row_q,
// row_q <- s row_p + c row_q.  Consecutive rotations mostly chain (p is the previous q), so the
// running row stays in a register and the q rows are loaded ahead, 8 rotations at a time.
__global__ __launch_bounds__(64) void k_dc_rot(const DcMerge *merges, const DcRot *rots) {
  const DcMerge M = merges[blockIdx.y];
  const int col = M.lo + blockIdx.x * 64 + threadIdx.x;
  if (M.nrot == 0 || col >= M.hi) return;
  const int half = col < M.m ? 1 : 2;
  double *zc = M.Zin + col;
  const int64_t ld = M.n;
  const DcRot *rt = rots + M.rot;
  int held = -1;  // row whose value `carry` is, not yet stored
  double carry = 0.0;
  constexpr int B = 8;
  for (int r0 = 0; r0 < M.nrot; r0 += B) {
    double qv[B];
#pragma unroll
    for (int b = 0; b < B; ++b) {
      qv[b] = 0.0;
      // a row is q of at most one rotation, and p only after that: no store in between changes it
      if (r0 + b < M.nrot && (rt[r0 + b].qf & half)) qv[b] = zc[rt[r0 + b].q * ld];
    }
#pragma unroll
    for (int b = 0; b < B; ++b) {
      if (r0 + b >= M.nrot) break;
      const DcRot R = rt[r0 + b];
      double a;
      if (R.p == held) {
        a = carry;
      } else {
        if (held >= 0) zc[held * ld] = carry;
        a = (R.pf & half) ? zc[R.p * ld] : 0.0;
      }
      zc[R.p * ld] = R.c * a - R.s * qv[b];
      carry = R.s * a + R.c * qv[b];
      held = R.q;
    }
  }
  if (held >= 0) zc[held * ld] = carry;
}

__global__ __launch_bounds__(kDcThreads) void k_dc_secular(const DcMerge *merges, DcRows rw) {
  const DcMerge M = merges[blockIdx.y];
  const int j = blockIdx.x * (kDcThreads / 64) + (threadIdx.x >> 6);
  if (j >= M.k) return;
  int org;
  double tau;
  secular_root(rw.pole + M.off, rw.z + M.off, M.k, M.rho, j, WaveLanes(), org, tau);
  if ((threadIdx.x & 63) == 0) {
    rw.org[M.off + j] = org;
    rw.tau[M.off + j] = tau;
  }
}

// zhat_i = sign(z_i) sqrt(prod_j (lam_j - d_i) / (rho prod_{j != i} (d_j - d_i)))  (Gu-Eisenstat),
// a wave per i; the ratios (lam_j - d_i) / (d_j - d_i) are of moderate size in any order.
__global__ __launch_bounds__(kDcThreads) void k_dc_zhat(const DcMerge *merges, DcRows rw) {
  const DcMerge M = merges[blockIdx.y];
  const int i = blockIdx.x * (kDcThreads / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (i >= M.k) return;
  const double *d = rw.pole + M.off, *tau = rw.tau + M.off;
  const int *org = rw.org + M.off;
  const double di = d[i];
  double p = 1.0;
  for (int j = lane; j < M.k; j += 64) {
    const double lmd = -((di - d[org[j]]) - tau[j]);  // lam_j - d_i
    p *= (j == i) ? lmd : lmd / (d[j] - di);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) p *= __shfl_xor(p, off, 64);
  if (lane == 0) {
    const double v = sqrt(fabs(p / M.rho));
    rw.zh[M.off + i] = (rw.z[M.off + i] >= 0.0) ? v : -v;
  }
}

// A wave per block row.  Row j < k: eigenvector j of the update, U[j][ucol(i)] = zhat_i / (d_i - lam_j)
// normalised, its eigenvalue and its place among the block's values (the roots and the deflated
// values are both ascending, so a binary search of the other list gives it).  Row k + t: deflated
// entry t, copied to its place, zero on the half its row is not supported on.
__global__ __launch_bounds__(kDcThreads) void k_dc_rows(const DcMerge *merges, DcRows rw) {
  const DcMerge M = merges[blockIdx.y];
  const int row = blockIdx.x * (kDcThreads / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int nb = M.hi - M.lo, k = M.k;
  if (row >= nb) return;
  const double *d = rw.pole + M.off, *tau = rw.tau + M.off, *zh = rw.zh + M.off, *dval = rw.dval + M.off;
  const int *org = rw.org + M.off;
  if (row < k) {
    const double dorg = d[org[row]], t = tau[row];
    double s = 0.0;
    for (int i = lane; i < k; i += 64) {
      const double u = zh[i] / ((d[i] - dorg) - t);
      s += u * u;
    }
    s = WaveLanes().sum(s);
    const double inv = 1.0 / sqrt(s);
    double *U = M.U + static_cast<int64_t>(M.lo + row) * M.n + M.lo;
    for (int i = lane; i < k; i += 64) U[rw.ucol[M.off + i]] = zh[i] / ((d[i] - dorg) - t) * inv;
    if (lane == 0) {
      const double lam = dorg + t;
      int a = 0, b = nb - k;  // deflated values <= lam
      while (a < b) {
        const int c = (a + b) >> 1;
        if (dval[c] <= lam) a = c + 1;
        else b = c;
      }
      rw.rank[M.off + row] = row + a;
      M.w[M.lo + row + a] = lam;
    }
    return;
  }
  const int t = row - k;
  const double v = dval[t];
  int a = 0, b = k;  // roots < v
  while (a < b) {
    const int c = (a + b) >> 1;
    if (d[org[c]] + tau[c] < v) a = c + 1;
    else b = c;
  }
  const int flag = rw.dflag[M.off + t];
  const double *src = M.Zin + static_cast<int64_t>(rw.dsrc[M.off + t]) * M.n;
  double *dst = M.Zout + static_cast<int64_t>(M.lo + t + a) * M.n;
  for (int c = M.lo + lane; c < M.hi; c += 64) dst[c] = (flag & (c < M.m ? 1 : 2)) ? src[c] : 0.0;
  if (lane == 0) M.w[M.lo + t + a] = v;
}

// G row q: the child row of U's column q, on the columns of the half or halves it is supported on.
__global__ __launch_bounds__(kDcThreads) void k_dc_gather(const DcMerge *merges, DcRows rw) {
  const DcMerge M = merges[blockIdx.y];
  const int q = blockIdx.x * (kDcThreads / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (q >= M.k) return;
  const int c0 = q < M.k12 ? M.lo : M.m, c1 = q >= M.k1 ? M.hi : M.m;
  const double *src = M.Zin + static_cast<int64_t>(rw.src[M.off + q]) * M.n;
  double *dst = M.G + static_cast<int64_t>(M.lo + q) * M.n;
  for (int c = c0 + lane; c < c1; c += 64) dst[c] = src[c];
}

// New rows = U G on each half's columns: the first half's need U's columns [0, k12) only, the second
// half's [k1, k).  blockIdx.y = 2 merge + half, blockIdx.x a 64 x 64 tile; a root's row goes to its
// place in the block (rank).  FP64 MFMA as in k_dgemm (same permuted-k LDS rows), but with 64 x 64
// tiles: a depth's products are a few hundred rows wide, and 128 x 128 tiles leave most of the
// compute units idle.
constexpr int kTB = 64, kTK = 16, kTS = 18;
__global__ __launch_bounds__(256) void k_dc_gemm(const DcMerge *merges, const int *rank) {
  __shared__ __attribute__((aligned(16))) double As[2][kTB][kTS];
  __shared__ __attribute__((aligned(16))) double Bs[2][kTB][kTS];
  const DcMerge M = merges[blockIdx.y >> 1];
  const int half = blockIdx.y & 1;
  const int cbeg = half ? M.m : M.lo, cend = half ? M.hi : M.m;
  const int kbeg = half ? M.k1 : 0, kend = half ? M.k : M.k12;
  const int nt = (cend - cbeg + kTB - 1) / kTB, mt = (M.k + kTB - 1) / kTB;
  if (static_cast<int>(blockIdx.x) >= nt * mt) return;
  const int tm = blockIdx.x / nt, tn = blockIdx.x - tm * nt;
  const int r0 = tm * kTB, c0 = cbeg + tn * kTB;
  const int64_t ld = M.n;
  const double *U = M.U + static_cast<int64_t>(M.lo) * ld + M.lo;
  const double *G = M.G + static_cast<int64_t>(M.lo) * ld;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
  // U slab: k = tid % 16 of rows tid / 16 + 16 q;  G slab: column tid % 64, k = (tid / 64) * 4 + q
  double ua[4], gb[4];
  const int uk = tid & 15, ur = tid >> 4, ukp = 4 * (uk & 3) + (uk >> 2);
  const int gc = tid & 63, gk = (tid >> 6) * 4;
  auto load = [&](int kb) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      ua[q] = (kb + uk < kend && r0 + ur + 16 * q < M.k) ? U[(r0 + ur + 16 * q) * ld + kb + uk] : 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      gb[q] = (kb + gk + q < kend && c0 + gc < cend) ? G[(kb + gk + q) * ld + c0 + gc] : 0.0;
  };
  auto store = [&](int buf) {
#pragma unroll
    for (int q = 0; q < 4; ++q) As[buf][ur + 16 * q][ukp] = ua[q];
    // k = gk + q, permuted 4 (k % 4) + k / 4 = 4 q + gk / 4
#pragma unroll
    for (int q = 0; q < 4; ++q) Bs[buf][gc][4 * q + (gk >> 2)] = gb[q];
  };
  v4d acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = v4d{0.0, 0.0, 0.0, 0.0};
  const int nk = kend > kbeg ? (kend - kbeg + kTK - 1) / kTK : 0;
  if (nk > 0) {
    load(kbeg);
    store(0);
  }
  __syncthreads();
  const int r = lane & 15, q4 = (lane >> 4) * 4;
  for (int kt = 0; kt < nk; ++kt) {
    const int buf = kt & 1;
    if (kt + 1 < nk) load(kbeg + (kt + 1) * kTK);
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
      v2d av[2], bv[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        av[i] = *reinterpret_cast<const v2d *>(&As[buf][wm + i * 16 + r][q4 + 2 * hf]);
        bv[i] = *reinterpret_cast<const v2d *>(&Bs[buf][wn + i * 16 + r][q4 + 2 * hf]);
      }
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[i][s2], bv[j][s2], acc[i][j], 0, 0, 0);
    }
    if (kt + 1 < nk) store(buf ^ 1);
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int row = r0 + wm + i * 16 + (lane >> 4) + 4 * e;
      if (row >= M.k) continue;
      double *out = M.Zout + static_cast<int64_t>(M.lo + rank[M.off + row]) * ld;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int c = c0 + wn + j * 16 + (lane & 15);
        if (c < cend) out[c] = acc[i][j][e];
      }
    }
}

inline unsigned nblk(int64_t n, int t) { return static_cast<unsigned>((n + t - 1) / t); }

// A node of the tree: the block [lo, hi) of one matrix at a depth.
struct Node {
  int job, lo, hi;
};

// Appends the nodes of [lo, hi) to the lists of their depths (halves of n / 2 and n - n / 2 rows
// until a block has at most kLeaf).
void plan_nodes(std::vector<std::vector<Node>> &inner, std::vector<std::vector<Node>> &leaf, int job, int lo, int hi,
                size_t depth) {
  if (inner.size() <= depth) {
    inner.resize(depth + 1);
    leaf.resize(depth + 1);
  }
  if (hi - lo <= kLeaf) {
    leaf[depth].push_back({job, lo, hi});
    return;
  }
  inner[depth].push_back({job, lo, hi});
  const int m = lo + (hi - lo) / 2;
  plan_nodes(inner, leaf, job, lo, m, depth + 1);
  plan_nodes(inner, leaf, job, m, hi, depth + 1);
}

size_t align8(size_t x) { return (x + 7) / 8 * 8; }

}  // namespace

size_t dc_work_doubles(int n) { return 3 * static_cast<size_t>(n) * n; }

dacp_status dc_tridiag_jobs(dacp_ctx ctx, const std::vector<DcJob> &jobs_in) {
  hipStream_t st = ctx->stream;
  std::vector<DcJob> jobs(jobs_in);
  std::vector<std::vector<Node>> inner, leaf;
  std::vector<size_t> woff(jobs.size() + 1, 0);
  for (size_t i = 0; i < jobs.size(); ++i) {
    woff[i + 1] = woff[i] + static_cast<size_t>(jobs[i].n);
    if (jobs[i].n > 0) plan_nodes(inner, leaf, static_cast<int>(i), 0, jobs[i].n, 0);
  }
  const size_t wtot = woff.back();
  if (wtot == 0) return DACP_OK;
  auto buffer = [&](int job, size_t depth) { return (depth & 1) ? jobs[job].work : jobs[job].Z; };

  size_t max_merges = 0, n_leaves = 0;
  for (const auto &v : inner) max_merges = std::max(max_merges, v.size());
  for (const auto &v : leaf) n_leaves += v.size();
  // device: eigenvalues and update vectors (copied to the host together, with the leaves' flag),
  // the depth's packed tables (one upload), and the kernels' own per-row arrays
  DevBuf wz, table, rows, dleaf;
  DACP_HIP(ctx, wz.alloc((2 * wtot + 1) * sizeof(double)));
  double *wdev = wz.as<double>(), *zdev = wdev + wtot;
  int *bad = reinterpret_cast<int *>(zdev + wtot);
  const size_t table_bytes = align8(max_merges * sizeof(DcMerge)) + align8(wtot * sizeof(DcRot)) +
                             3 * wtot * sizeof(double) + 4 * align8(wtot * sizeof(int));
  DACP_HIP(ctx, table.alloc(table_bytes));
  DACP_HIP(ctx, rows.alloc(2 * wtot * sizeof(double) + 2 * align8(wtot * sizeof(int))));
  DACP_HIP(ctx, dleaf.alloc(n_leaves * sizeof(DcLeaf)));

  // the diagonals come to the host once: the tears' weights and a check that they are finite
  std::vector<double> eh(wtot, 0.0), dh(wtot, 0.0);
  for (size_t i = 0; i < jobs.size(); ++i) {
    if (jobs[i].n <= 0) continue;
    DACP_HIP(ctx, hipMemcpyAsync(dh.data() + woff[i], jobs[i].d, jobs[i].n * sizeof(double), hipMemcpyDeviceToHost, st));
    if (jobs[i].n > 1)
      DACP_HIP(ctx, hipMemcpyAsync(eh.data() + woff[i], jobs[i].e, (jobs[i].n - 1) * sizeof(double),
                                   hipMemcpyDeviceToHost, st));
  }
  // the merges' blocks and buffers, every depth in one upload (the update vectors' kernel reads them)
  std::vector<DcMerge> geo;
  std::vector<size_t> geo_at(inner.size());
  for (size_t depth = 0; depth < inner.size(); ++depth) {
    geo_at[depth] = geo.size();
    int off = 0;
    for (const Node &nd : inner[depth]) {
      const DcJob &jb = jobs[nd.job];
      const size_t nn = static_cast<size_t>(jb.n) * jb.n;
      DcMerge M;
      std::memset(&M, 0, sizeof(M));
      M.Zin = buffer(nd.job, depth + 1);
      M.Zout = buffer(nd.job, depth);
      M.U = jb.work + nn;
      M.G = jb.work + 2 * nn;
      M.w = wdev + woff[nd.job];
      M.n = jb.n;
      M.lo = nd.lo;
      M.hi = nd.hi;
      M.m = nd.lo + (nd.hi - nd.lo) / 2;
      M.off = off;
      off += nd.hi - nd.lo;
      geo.push_back(M);
    }
  }
  DevBuf dgeo;
  DACP_HIP(ctx, dgeo.alloc(geo.size() * sizeof(DcMerge)));
  DACP_TRY(to_device(ctx, dgeo.p, geo.data(), geo.size() * sizeof(DcMerge)));
  if (geo.empty()) DACP_HIP(ctx, hipStreamSynchronize(st));  // else the upload has waited for the diagonals
  for (size_t i = 0; i < wtot; ++i)
    if (!std::isfinite(dh[i]) || !std::isfinite(eh[i]))
      return set_err(ctx, DACP_E_NUMERIC, "divide and conquer: non-finite tridiagonal entry");
  // A matrix of a scale far from 1 is solved as its multiple by a power of two (which is exact): the secular
  // equation squares the poles' distances and their reciprocals.
  std::vector<int> scale(jobs.size(), 0);
  DevBuf scaled;
  {
    size_t at = 0;
    for (size_t i = 0; i < jobs.size(); ++i) {
      double top = 0.0;
      for (size_t q = woff[i]; q < woff[i + 1]; ++q) top = std::max({top, std::fabs(dh[q]), std::fabs(eh[q])});
      if (top > 0.0 && (top < 1e-60 || top > 1e60)) scale[i] = std::ilogb(top), at += 2 * static_cast<size_t>(jobs[i].n);
    }
    if (at > 0) {
      std::vector<double> host;
      DACP_HIP(ctx, scaled.alloc(at * sizeof(double)));
      for (size_t i = 0; i < jobs.size(); ++i) {
        if (scale[i] == 0) continue;
        for (std::vector<double> *v : {&dh, &eh}) {
          (v == &dh ? jobs[i].d : jobs[i].e) = scaled.as<double>() + host.size();
          for (size_t q = woff[i]; q < woff[i + 1]; ++q) host.push_back((*v)[q] = std::scalbn((*v)[q], -scale[i]));
        }
      }
      DACP_TRY(to_device(ctx, scaled.p, host.data(), at * sizeof(double)));
    }
  }
  {
    std::vector<DcLeaf> ls;
    for (size_t t = 0; t < leaf.size(); ++t)
      for (const Node &nd : leaf[t])
        ls.push_back({jobs[nd.job].d, jobs[nd.job].e, buffer(nd.job, t), wdev + woff[nd.job], jobs[nd.job].n, nd.lo, nd.hi});
    const int zero = 0;
    DACP_HIP(ctx, hipMemcpyAsync(bad, &zero, sizeof(int), hipMemcpyHostToDevice, st));
    DACP_TRY(to_device(ctx, dleaf.p, ls.data(), ls.size() * sizeof(DcLeaf)));
    hipLaunchKernelGGL(k_dc_leaf, dim3(static_cast<unsigned>(ls.size())), dim3(64), 0, st, dleaf.as<DcLeaf>(), bad);
    DACP_HIP(ctx, hipGetLastError());
  }

  std::vector<double> host_wz(2 * wtot + 1);
  std::vector<unsigned char> blob(table_bytes);
  std::vector<DcMerge> ms;
  for (size_t depth = inner.size(); depth-- > 0;) {
    const std::vector<Node> &nodes = inner[depth];
    if (nodes.empty()) continue;
    ms.assign(geo.begin() + geo_at[depth], geo.begin() + geo_at[depth] + nodes.size());
    int off = 0, max_n = 0;
    for (const DcMerge &M : ms) {
      off += M.hi - M.lo;
      max_n = std::max(max_n, M.hi - M.lo);
    }
    const unsigned nm = static_cast<unsigned>(ms.size());
    hipLaunchKernelGGL(k_dc_z, dim3(nblk(max_n, 256), nm), dim3(256), 0, st, dgeo.as<DcMerge>() + geo_at[depth], zdev);
    DACP_HIP(ctx, hipGetLastError());
    DACP_TRY(to_host(ctx, host_wz.data(), wdev, (2 * wtot + 1) * sizeof(double)));
    int failed = 0;
    std::memcpy(&failed, host_wz.data() + 2 * wtot, sizeof(int));
    if (failed) return set_err(ctx, DACP_E_CONVERGENCE, "divide and conquer: leaf QR did not converge");

    // deflation of every merge (host_rules.cpp), packed for one upload
    size_t at = align8(nm * sizeof(DcMerge));
    const size_t arr = static_cast<size_t>(off);
    auto carve = [&](size_t bytes) {
      const size_t p = at;
      at += align8(bytes);
      return p;
    };
    const size_t o_pole = carve(arr * sizeof(double)), o_z = carve(arr * sizeof(double)),
                 o_dval = carve(arr * sizeof(double)), o_ucol = carve(arr * sizeof(int)),
                 o_src = carve(arr * sizeof(int)), o_dsrc = carve(arr * sizeof(int)), o_dflag = carve(arr * sizeof(int)),
                 o_rot = at;
    double *pole = reinterpret_cast<double *>(blob.data() + o_pole), *zv = reinterpret_cast<double *>(blob.data() + o_z),
           *dval = reinterpret_cast<double *>(blob.data() + o_dval);
    int *ucol = reinterpret_cast<int *>(blob.data() + o_ucol), *src = reinterpret_cast<int *>(blob.data() + o_src),
        *dsrc = reinterpret_cast<int *>(blob.data() + o_dsrc), *dflag = reinterpret_cast<int *>(blob.data() + o_dflag);
    DcRot *rots = reinterpret_cast<DcRot *>(blob.data() + o_rot);
    int nrot = 0, max_k = 0;
    std::vector<int> flag, dorder;
    // the merges' deflations are independent: over host threads when there is work for them
    std::vector<rules::DcDeflation> dfs(nodes.size());
    auto deflate = [&](int i) {
      DcMerge &M = ms[i];
      const int n = M.hi - M.lo, n1 = M.m - M.lo;
      const double beta = eh[woff[nodes[i].job] + M.m - 1];
      std::vector<double> z(host_wz.begin() + wtot + M.off, host_wz.begin() + wtot + M.off + n);
      const double *wv = host_wz.data() + woff[nodes[i].job] + M.lo;
      std::vector<double> dv(wv, wv + n);
      // T = diag(T1, T2) torn + |beta| v v^T, v = (sign(beta) e_last; e_first); z normalised, rho
      // absorbs |z|^2
      double zn = 0.0;
      for (int q = 0; q < n; ++q) {
        if (q < n1 && beta < 0.0) z[q] = -z[q];
        zn += z[q] * z[q];
      }
      if (!std::isfinite(zn) || !(zn > 0.0)) {
        M.rho = NAN;
        return;
      }
      zn = std::sqrt(zn);
      for (double &x : z) x /= zn;
      M.rho = std::fabs(beta) * zn * zn;
      dfs[i] = rules::dc_deflate(dv, z, M.rho, M.lo);
    };
    host_parallel(static_cast<int>(nodes.size()), std::min(ctx->batch_workers, off / 4096), deflate);
    for (size_t i = 0; i < nodes.size(); ++i) {
      DcMerge &M = ms[i];
      const int n = M.hi - M.lo, n1 = M.m - M.lo;
      if (std::isnan(M.rho)) return set_err(ctx, DACP_E_NUMERIC, "divide and conquer: non-finite update vector");
      const rules::DcDeflation &df = dfs[i];
      // halves each row is supported on: its own, both once a rotation has mixed it
      flag.assign(n, 0);
      for (int q = 0; q < n; ++q) flag[q] = q < n1 ? 1 : 2;
      M.rot = nrot;
      M.nrot = static_cast<int>(df.rot_cs.size() / 2);
      for (int q = 0; q < M.nrot; ++q) {
        DcRot &R = rots[nrot++];
        R.c = df.rot_cs[2 * q];
        R.s = df.rot_cs[2 * q + 1];
        R.p = df.rot_pq[2 * q];
        R.q = df.rot_pq[2 * q + 1];
        int &fp = flag[R.p - M.lo], &fq = flag[R.q - M.lo];
        R.pf = fp;
        R.qf = fq;
        fp = fq = fp | fq;
      }
      M.k = static_cast<int>(df.nd.size());
      max_k = std::max(max_k, M.k);
      int cnt[4] = {0, 0, 0, 0};
      for (int j : df.nd) ++cnt[flag[df.rowid[j] - M.lo]];
      M.k1 = cnt[1];
      M.k12 = cnt[1] + cnt[3];
      int next[4] = {0, 0, cnt[1] + cnt[3], cnt[1]};  // next column of the rows on half 1 / half 2 / both
      for (int q = 0; q < M.k; ++q) {
        const int j = df.nd[q], row = df.rowid[j];
        const int c = next[flag[row - M.lo]]++;
        pole[M.off + q] = df.ds[j];
        zv[M.off + q] = df.zs[j];
        ucol[M.off + q] = c;
        src[M.off + c] = row;
      }
      dorder.clear();
      for (int j = 0; j < n; ++j)
        if (df.defl[j]) dorder.push_back(j);
      std::stable_sort(dorder.begin(), dorder.end(), [&](int a, int b) { return df.ds[a] < df.ds[b]; });
      for (size_t t = 0; t < dorder.size(); ++t) {
        dval[M.off + t] = df.ds[dorder[t]];
        dsrc[M.off + t] = df.rowid[dorder[t]];
        dflag[M.off + t] = flag[df.rowid[dorder[t]] - M.lo];
      }
    }
    std::memcpy(blob.data(), ms.data(), nm * sizeof(DcMerge));
    DACP_TRY(to_device(ctx, table.p, blob.data(), o_rot + nrot * sizeof(DcRot)));
    const unsigned char *tb = table.as<unsigned char>();
    const DcMerge *dm = table.as<DcMerge>();
    DcRows rw;
    rw.pole = reinterpret_cast<const double *>(tb + o_pole);
    rw.z = reinterpret_cast<const double *>(tb + o_z);
    rw.dval = reinterpret_cast<const double *>(tb + o_dval);
    rw.ucol = reinterpret_cast<const int *>(tb + o_ucol);
    rw.src = reinterpret_cast<const int *>(tb + o_src);
    rw.dsrc = reinterpret_cast<const int *>(tb + o_dsrc);
    rw.dflag = reinterpret_cast<const int *>(tb + o_dflag);
    rw.tau = rows.as<double>();
    rw.zh = rw.tau + wtot;
    rw.org = reinterpret_cast<int *>(rw.zh + wtot);
    rw.rank = rw.org + align8(wtot * sizeof(int)) / sizeof(int);
    if (nrot > 0) {
      hipLaunchKernelGGL(k_dc_rot, dim3(nblk(max_n, 64), nm), dim3(64), 0, st, dm,
                         reinterpret_cast<const DcRot *>(tb + o_rot));
      DACP_HIP(ctx, hipGetLastError());
    }
    const int per = kDcThreads / 64;
    if (max_k > 0) {
      hipLaunchKernelGGL(k_dc_secular, dim3(nblk(max_k, per), nm), dim3(kDcThreads), 0, st, dm, rw);
      hipLaunchKernelGGL(k_dc_zhat, dim3(nblk(max_k, per), nm), dim3(kDcThreads), 0, st, dm, rw);
      hipLaunchKernelGGL(k_dc_gather, dim3(nblk(max_k, per), nm), dim3(kDcThreads), 0, st, dm, rw);
      DACP_HIP(ctx, hipGetLastError());
    }
    hipLaunchKernelGGL(k_dc_rows, dim3(nblk(max_n, per), nm), dim3(kDcThreads), 0, st, dm, rw);
    DACP_HIP(ctx, hipGetLastError());
    if (max_k > 0) {
      const unsigned tiles = nblk(max_k, kTB) * nblk((max_n + 1) / 2, kTB);
      hipLaunchKernelGGL(k_dc_gemm, dim3(tiles, 2 * nm), dim3(256), 0, st, dm, rw.rank);
      DACP_HIP(ctx, hipGetLastError());
    }
  }
  DACP_TRY(to_host(ctx, host_wz.data(), wdev, (2 * wtot + 1) * sizeof(double)));
  int failed = 0;
  std::memcpy(&failed, host_wz.data() + 2 * wtot, sizeof(int));
  if (failed) return set_err(ctx, DACP_E_CONVERGENCE, "divide and conquer: leaf QR did not converge");
  for (size_t i = 0; i < wtot; ++i)
    if (!std::isfinite(host_wz[i])) return set_err(ctx, DACP_E_NUMERIC, "divide and conquer: non-finite root");
  for (size_t i = 0; i < jobs.size(); ++i)
    for (int q = 0; q < jobs[i].n; ++q) jobs[i].w[q] = std::scalbn(host_wz[woff[i] + q], scale[i]);
  return DACP_OK;
}

}  // namespace dacp
