// FP64 GEMM on the gfx950 matrix cores (v_mfma_f64_16x16x4_f64).
//
// C = alpha * op(A) * op(B) + beta * C, row-major.  A 256-thread workgroup
// computes a 128 x 128 tile of C (64 x 64 for small outputs); each of its four
// 64-lane waves owns a quadrant held as 4 x 4 (2 x 2) MFMA accumulators of
// 16 x 16.  K advances in slabs of 16 staged through double-buffered LDS.
// Used for the Gram S = V^T V and P = V^T (H V) (upper triangle only), the
// subspace transforms of the generalised eigenproblem and the Ritz vectors.
//
// LDS layout.  The 16 x 16 x 4 MFMA takes from lane l the A element (row l % 16, k = l / 16) and
// the B element (k = l / 16, column l % 16), so over the four k-steps of a slab lane l needs
// k = l / 16 + 4 s, s = 0..3, of one row.  Each operand tile is stored row-major by m (or n) with
// the slab's k permuted as kp(k) = 4 (k % 4) + k / 4: those four values are contiguous, and a
// lane fetches them with two 16-byte LDS reads.  Rows are 18 doubles (144 bytes) apart, so the 16
// lanes of a read group hit distinct 16-byte bank groups.
#include <hip/hip_runtime.h>

#include "internal.h"

namespace dacp {

typedef double v4d __attribute__((ext_vector_type(4)));
typedef double v2d __attribute__((ext_vector_type(2)));

constexpr int BK = 16, KS = 18;
constexpr int kBand = 8;  // tile rows walked together (see tile_at)

// Global -> registers -> LDS staging of one TM x 16 operand slab by 256 threads.  KMAJOR: element
// (k, x) at src[k * ld + x] (x = m or n contiguous); each thread takes one x and NV consecutive k.
// Otherwise element (k, x) at src[x * ld + k]; each thread takes one k and NV rows x.
template <bool KMAJOR, int TM>
struct Slab {
  static constexpr int NV = TM / 16;
  double v[NV];
  // Row q of the thread's NV starts at a wave-uniform pointer (KMAJOR: k is uniform per wave) or at
  // a uniform pointer plus one per-lane offset computed once, so the loads need no per-element
  // 64-bit address registers.
  __device__ __forceinline__ void load(const double *src, int64_t ld, int64_t x0, int64_t X, int64_t kb, int64_t kend,
                                       int tid) {
    if (KMAJOR) {
      const int x = tid & (TM - 1), kk = (tid / TM) * NV;
      const bool xin = x0 + x < X;
      const double *base = src + (kb + kk) * ld + x0;
#pragma unroll
      for (int q = 0; q < NV; ++q) v[q] = (kb + kk + q < kend && xin) ? base[q * ld + x] : 0.0;
    } else {
      const int k = tid & 15, xr = tid >> 4;
      const bool kin = kb + k < kend;
      const int64_t off = static_cast<int64_t>(xr) * ld + k;
      const double *base = src + x0 * ld + kb;
#pragma unroll
      for (int q = 0; q < NV; ++q)
        v[q] = (kin && x0 + xr + 16 * q < X) ? base[static_cast<int64_t>(16 * q) * ld + off] : 0.0;
    }
  }
  __device__ __forceinline__ void store(double (*S)[KS], int tid) const {
    if (KMAJOR) {
      const int x = tid & (TM - 1), h = tid / TM;
      if constexpr (NV == 8) {
        // k = 8 h + c and k + 4 are adjacent after the permutation
#pragma unroll
        for (int c = 0; c < 4; ++c) *reinterpret_cast<v2d *>(&S[x][4 * c + 2 * h]) = v2d{v[c], v[c + 4]};
      } else {
#pragma unroll
        for (int c = 0; c < NV; ++c) S[x][4 * c + h] = v[c];
      }
    } else {
      const int k = tid & 15, kp = 4 * (k & 3) + (k >> 2);
#pragma unroll
      for (int q = 0; q < NV; ++q) S[(tid >> 4) + 16 * q][kp] = v[q];
    }
  }
};

// Number of output tiles of a grid of ntm x ntn tiles (upper: those with tile row <= tile column,
// ntm == ntn), and tile number t of the walk: bands of kBand tile rows, column by column inside a
// band, so that any 64 consecutive tiles are close to an 8 x 8 block, which shares 8 row panels of
// op(A) and 8 column panels of op(B).
__host__ __device__ inline int64_t tile_count(int ntm, int ntn, int upper) {
  return upper ? static_cast<int64_t>(ntn) * (ntn + 1) / 2 : static_cast<int64_t>(ntm) * ntn;
}
__device__ __forceinline__ void tile_at(int t, int ntm, int ntn, int upper, int &tm, int &tn) {
  if (!upper) {
    const int band = t / (kBand * ntn), r = t - band * kBand * ntn;
    const int h = min(kBand, ntm - band * kBand);
    tn = r / h;
    tm = band * kBand + (r - tn * h);
    return;
  }
  int r0 = 0, h = min(kBand, ntn);
  for (;;) {  // a band's triangle (h (h + 1) / 2 tiles), then its full columns
    const int n = h * (h + 1) / 2 + (ntn - r0 - h) * h;
    if (t < n) break;
    t -= n;
    r0 += kBand;
    h = min(kBand, ntn - r0);
  }
  int c = 0;
  while (c < h && t >= c + 1) {
    t -= c + 1;
    ++c;
  }
  if (c == h) {
    c += t / h;
    t -= (c - h) * h;
  }
  tm = r0 + t;
  tn = r0 + c;
}

// Workgroups are dealt to the 8 XCDs round-robin, workgroup 8 q + x to XCD x.  Work unit u is tile
// u mod ntiles of K range u / ntiles, and each XCD takes a contiguous eighth of the units in order:
// its resident workgroups then walk neighbouring tiles of one K range (which its L2 holds), and
// all XCDs carry the same load whatever the number of tiles.  (Dealing whole rounds of 64 tiles to
// an XCD left 5 of the 8 idle on a 15 x 15 grid of tiles: V^T V at D = 2^17, m = 1873 took 36.8 ms.)
// Split K: range z covers k in [z kchunk, (z + 1) kchunk); with `work` set, alpha times its partial
// tile goes to work[z][M][N] for k_splitk_reduce.
template <int TA, int TB, int TM>
__global__ __launch_bounds__(256, 2) void k_dgemm(int64_t M, int64_t N, int64_t K, double alpha, const double *A,
                                                  int64_t lda, const double *B, int64_t ldb, double beta, double *C,
                                                  int64_t ldc, int upper, int ntm, int ntn, int64_t kchunk,
                                                  int64_t units, double *work) {
  constexpr int F = TM / 32;  // 16 x 16 accumulators per wave and dimension: four waves in a 2 x 2 grid
  __shared__ __attribute__((aligned(16))) double As[2][TM][KS];
  __shared__ __attribute__((aligned(16))) double Bs[2][TM][KS];
  const int64_t x = blockIdx.x & 7, q = blockIdx.x >> 3;
  const int64_t ubeg = x * units / 8, uend = (x + 1) * units / 8;
  if (ubeg + q >= uend) return;
  const int ntiles = static_cast<int>(tile_count(ntm, ntn, upper));
  const int64_t z = (ubeg + q) / ntiles;
  int tm, tn;
  tile_at(static_cast<int>(ubeg + q - z * ntiles), ntm, ntn, upper, tm, tn);
  const int64_t m0 = static_cast<int64_t>(tm) * TM;
  const int64_t n0 = static_cast<int64_t>(tn) * TM;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = (wave >> 1) * (TM / 2);
  const int wn = (wave & 1) * (TM / 2);

  const int64_t kbeg = z * kchunk;
  const int64_t kend = (kbeg + kchunk < K) ? kbeg + kchunk : K;
  Slab<TA == 1, TM> sa;   // A stored K x M when transposed
  Slab<TB == 0, TM> sbt;  // B stored K x N when not transposed

  v4d acc[F][F];
#pragma unroll
  for (int i = 0; i < F; ++i)
#pragma unroll
    for (int j = 0; j < F; ++j) acc[i][j] = v4d{0.0, 0.0, 0.0, 0.0};

  const int64_t nk = (kend > kbeg) ? (kend - kbeg + BK - 1) / BK : 0;
  sa.load(A, lda, m0, M, kbeg, kend, tid);
  sbt.load(B, ldb, n0, N, kbeg, kend, tid);
  sa.store(As[0], tid);
  sbt.store(Bs[0], tid);
  __syncthreads();
  const int r = lane & 15, q4 = (lane >> 4) * 4;
  for (int64_t kt = 0; kt < nk; ++kt) {
    const int buf = static_cast<int>(kt & 1);
    if (kt + 1 < nk) {
      sa.load(A, lda, m0, M, kbeg + (kt + 1) * BK, kend, tid);
      sbt.load(B, ldb, n0, N, kbeg + (kt + 1) * BK, kend, tid);
    }
    // two k-steps per 16-byte read: halves 0 (k-steps 0, 1) and 1 (k-steps 2, 3) of the slab
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
      v2d av[F], bv[F];
#pragma unroll
      for (int i = 0; i < F; ++i) {
        av[i] = *reinterpret_cast<const v2d *>(&As[buf][wm + i * 16 + r][q4 + 2 * hf]);
        bv[i] = *reinterpret_cast<const v2d *>(&Bs[buf][wn + i * 16 + r][q4 + 2 * hf]);
      }
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
        for (int i = 0; i < F; ++i)
#pragma unroll
          for (int j = 0; j < F; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[i][s2], bv[j][s2], acc[i][j], 0, 0, 0);
    }
    if (kt + 1 < nk) {
      sa.store(As[buf ^ 1], tid);
      sbt.store(Bs[buf ^ 1], tid);
    }
    __syncthreads();
  }
  // Output layout of the f64 16x16 accumulator (measured on gfx950): lane l,
  // item r -> row (l / 16) + 4 r, column l % 16.
#pragma unroll
  for (int i = 0; i < F; ++i)
#pragma unroll
    for (int j = 0; j < F; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int64_t row = m0 + wm + i * 16 + (lane >> 4) + 4 * e;
        const int64_t col = n0 + wn + j * 16 + (lane & 15);
        if (row < M && col < N) {
          double v = alpha * acc[i][j][e];
          if (work) {
            work[z * M * N + row * N + col] = v;
          } else {
            if (beta != 0.0) v += beta * C[row * ldc + col];
            C[row * ldc + col] = v;
          }
        }
      }
}

// C = sum_z work[z] + beta C (fixed order over z); upper: only the tiles (of 128) on or above the
// diagonal, the others' work is not written.
__global__ void k_splitk_reduce(const double *work, int splits, int64_t M, int64_t N, double beta, double *C,
                                int64_t ldc, int upper) {
  const int64_t e = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (e >= M * N) return;
  const int64_t row = e / N, col = e - row * N;
  if (upper && row / 128 > col / 128) return;
  double v = 0.0;
  for (int z = 0; z < splits; ++z) v += work[static_cast<int64_t>(z) * M * N + e];
  if (beta != 0.0) v += beta * C[row * ldc + col];
  C[row * ldc + col] = v;
}

template <int TM>
static hipError_t launch_dgemm_tm(int transA, int transB, int64_t M, int64_t N, int64_t K, double alpha,
                                  const double *A, int64_t lda, const double *B, int64_t ldb, double beta, double *C,
                                  int64_t ldc, int upper, int splits, double *work, hipStream_t s) {
  const int64_t tmc = (M + TM - 1) / TM, tnc = (N + TM - 1) / TM;
  const int64_t units = tile_count(static_cast<int>(tmc), static_cast<int>(tnc), upper) * splits;
  const int64_t nblocks = 8 * ((units + 7) / 8);
  if (tmc > 0x7fffffff || tnc > 0x7fffffff / kBand || nblocks > 0x7fffffff) return hipErrorInvalidValue;
  const int64_t kchunk = splits == 1 ? K : ((K + splits - 1) / splits + BK - 1) / BK * BK;
  double *wk = splits > 1 ? work : nullptr;
#define DACP_GEMM_LAUNCH(a_, b_)                                                                                     \
  hipLaunchKernelGGL((k_dgemm<a_, b_, TM>), dim3(static_cast<unsigned>(nblocks)), dim3(256), 0, s, M, N, K, alpha, A, \
                     lda, B, ldb, beta, C, ldc, upper, static_cast<int>(tmc), static_cast<int>(tnc), kchunk, units, wk)
  if (!transA && !transB) DACP_GEMM_LAUNCH(0, 0);
  else if (!transA && transB) DACP_GEMM_LAUNCH(0, 1);
  else if (transA && !transB) DACP_GEMM_LAUNCH(1, 0);
  else DACP_GEMM_LAUNCH(1, 1);
#undef DACP_GEMM_LAUNCH
  return hipGetLastError();
}

hipError_t launch_dgemm_impl(int transA, int transB, int64_t M, int64_t N, int64_t K, double alpha, const double *A,
                             int64_t lda, const double *B, int64_t ldb, double beta, double *C, int64_t ldc,
                             int upper, int splits, double *work, hipStream_t s) {
  if (M <= 0 || N <= 0) return hipSuccess;
  if (splits < 1 || (splits > 1 && !work)) return hipErrorInvalidValue;
  if (upper && M != N) return hipErrorInvalidValue;
  // 64 x 64 tiles when 128 x 128 ones would leave compute units without a workgroup (they reach about
  // two thirds of the large tiles' rate, on four times as many units) or be half empty.
  const int64_t t128 = tile_count(static_cast<int>((M + 127) / 128), static_cast<int>((N + 127) / 128), upper) * splits;
  hipError_t e;
  if ((splits == 1 && t128 < 256) || M <= 64 || N <= 64)
    e = launch_dgemm_tm<64>(transA, transB, M, N, K, alpha, A, lda, B, ldb, beta, C, ldc, upper, splits, work, s);
  else
    e = launch_dgemm_tm<128>(transA, transB, M, N, K, alpha, A, lda, B, ldb, beta, C, ldc, upper, splits, work, s);
  if (e != hipSuccess || splits == 1) return e;
  hipLaunchKernelGGL(k_splitk_reduce, dim3(static_cast<unsigned>((M * N + 255) / 256)), dim3(256), 0, s, work, splits,
                     M, N, beta, C, ldc, upper);
  return hipGetLastError();
}

// K ranges for a product of 128 x 128 tiles, at least min_rows deep each: the count whose rounds of
// two workgroups per compute unit take the least time, a range costing its depth plus 256 rows'
// worth of start and end, plus the partial tiles' write and read (one element's 16 bytes at about
// 4 TB/s against one row of a tile at the CU's share of 60 TFLOP/s).
int gemm_splits(int64_t M, int64_t N, int64_t K, int upper, int cus, int64_t min_rows, int max_splits) {
  const int64_t t = tile_count(static_cast<int>((M + 127) / 128), static_cast<int>((N + 127) / 128), upper);
  const int64_t slots = 2 * static_cast<int64_t>(cus);
  int best = 1;
  double best_cost = 0.0;
  for (int sp = 1; sp <= max_splits; ++sp) {
    if (sp > 1 && K / sp < min_rows) break;
    const double rounds = static_cast<double>((t * sp + slots - 1) / slots);
    const double per_row = 32768.0 * slots / 60e12;
    double cost = rounds * (static_cast<double>(K) / sp + 256.0) * per_row;
    if (sp > 1) cost += 16.0 * sp * static_cast<double>(M) * N * (upper ? 0.5 : 1.0) / 4e12 + 5e-6;
    if (sp == 1 || cost < 0.97 * best_cost) {
      best = sp;
      best_cost = cost;
    }
  }
  return best;
}

hipError_t launch_dgemm(int transA, int transB, int64_t M, int64_t N, int64_t K, double alpha, const double *A,
                        int64_t lda, const double *B, int64_t ldb, double beta, double *C, int64_t ldc, int upper,
                        hipStream_t s) {
  return launch_dgemm_impl(transA, transB, M, N, K, alpha, A, lda, B, ldb, beta, C, ldc, upper, 1, nullptr, s);
}

// With upper set (M == N), only tiles on or above the diagonal are computed and the reduction
// leaves the tiles below it undefined: the caller mirrors the upper triangle afterwards.
hipError_t launch_dgemm_splitk(int transA, int transB, int64_t M, int64_t N, int64_t K, double alpha, const double *A,
                               int64_t lda, const double *B, int64_t ldb, double beta, double *C, int64_t ldc,
                               int upper, int splits, double *work, hipStream_t s) {
  return launch_dgemm_impl(transA, transB, M, N, K, alpha, A, lda, B, ldb, beta, C, ldc, upper, splits, work, s);
}

// Copy the upper triangle onto the lower one (tiled through LDS).
__global__ void k_mirror_upper(double *C, int64_t n, int64_t ldc) {
  __shared__ double t[32][33];
  const int64_t bi = blockIdx.y, bj = blockIdx.x;
  if (bi > bj) return;  // source tile (bi, bj) in the upper part
  const int tx = threadIdx.x, ty = threadIdx.y;
  for (int r = ty; r < 32; r += 8) {
    const int64_t i = bi * 32 + r, j = bj * 32 + tx;
    t[r][tx] = (i < n && j < n) ? C[i * ldc + j] : 0.0;
  }
  __syncthreads();
  for (int r = ty; r < 32; r += 8) {
    const int64_t i = bj * 32 + r, j = bi * 32 + tx;  // destination (row i, col j) = source (j, i)
    if (i < n && j < n && i > j) C[i * ldc + j] = t[tx][r];
  }
}

hipError_t launch_mirror_upper(double *C, int64_t n, int64_t ldc, hipStream_t s) {
  const unsigned nt = static_cast<unsigned>((n + 31) / 32);
  hipLaunchKernelGGL(k_mirror_upper, dim3(nt, nt), dim3(32, 8), 0, s, C, n, ldc);
  return hipGetLastError();
}

// C <- (C + C^T) / 2, tile pairs handled by the upper tile's workgroup.
__global__ void k_symmetrize(double *C, int64_t n, int64_t ldc) {
  __shared__ double tu[32][33], tl[32][33];
  const int64_t bi = blockIdx.y, bj = blockIdx.x;
  if (bi > bj) return;
  const int tx = threadIdx.x, ty = threadIdx.y;
  for (int r = ty; r < 32; r += 8) {
    const int64_t i = bi * 32 + r, j = bj * 32 + tx;
    tu[r][tx] = (i < n && j < n) ? C[i * ldc + j] : 0.0;
    const int64_t i2 = bj * 32 + r, j2 = bi * 32 + tx;
    tl[r][tx] = (i2 < n && j2 < n) ? C[i2 * ldc + j2] : 0.0;
  }
  __syncthreads();
  for (int r = ty; r < 32; r += 8) {
    const int64_t i = bi * 32 + r, j = bj * 32 + tx;
    const double v = 0.5 * (tu[r][tx] + tl[tx][r]);
    if (i < n && j < n) C[i * ldc + j] = v;
    const int64_t i2 = bj * 32 + r, j2 = bi * 32 + tx;
    const double v2 = 0.5 * (tl[r][tx] + tu[tx][r]);
    if (i2 < n && j2 < n && bi != bj) C[i2 * ldc + j2] = v2;
  }
}

hipError_t launch_symmetrize(double *C, int64_t n, int64_t ldc, hipStream_t s) {
  const unsigned nt = static_cast<unsigned>((n + 31) / 32);
  hipLaunchKernelGGL(k_symmetrize, dim3(nt, nt), dim3(32, 8), 0, s, C, n, ldc);
  return hipGetLastError();
}

}  // namespace dacp
