// Dense symmetric eigensolver for matrices of up to 3072 rows, one or many at once (App. C's two
// eigen-decompositions): Householder tridiagonalisation with the matrix held in registers across
// the GPU, divide and conquer on the tridiagonals (dc.hip), and the reflectors applied to the
// eigenvectors in compact WY blocks.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <numeric>
#include <vector>

#include "internal.h"
#include "wave.h"

namespace dacp {

namespace {

constexpr unsigned long long kEmpty = ~0ull;  // exchange slot not written yet

// One matrix of a launch: workgroups wg0 .. wg0 + G - 1 hold its rows.
struct TriProb {
  const double *A;  // n x n, row stride lda, symmetric; read only
  int64_t lda;
  double *V;        // n x n: row k = the k-th reflector's vector, zero at columns <= k
  double *X;        // exchange, 2 n doubles per step, filled with kEmpty
  double *d, *e, *beta;
  int n, G, wg0;
};

// Four values a lane, each summed over the wave: two lane-half swaps pack them into one register, 16
// lanes each, which four DPP steps then add; the lanes of 16 h .. 16 h + 15 end with the sum of
// a[packed_row(h)].
__device__ __forceinline__ double wave_sum_4(double (&a)[4]) {
  auto swap32 = [](double &x, double &y) {
    const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(x), __double2loint(y), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(x), __double2hiint(y), false, false);
    x = __hiloint2double(hi[0], lo[0]);
    y = __hiloint2double(hi[1], lo[1]);
  };
  auto swap16 = [](double &x, double &y) {
    const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(x), __double2loint(y), false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(x), __double2hiint(y), false, false);
    x = __hiloint2double(hi[0], lo[0]);
    y = __hiloint2double(hi[1], lo[1]);
  };
  swap32(a[0], a[1]);
  swap32(a[2], a[3]);
  double u = a[0] + a[1], v = a[2] + a[3];
  swap16(u, v);
  double t = u + v;
  t += dpp_move<0xB1, 0xf>(t);
  t += dpp_move<0x4E, 0xf>(t);
  t += dpp_move<0x141, 0xf>(t);
  t += dpp_move<0x140, 0xf>(t);
  return t;
}
__device__ __forceinline__ int packed_row(int h) { return ((h & 1) << 1) | (h >> 1); }

__device__ __forceinline__ void publish(double *slot, double v) {
  unsigned long long b = __double_as_longlong(v);
  if (b == kEmpty) b = 0x7ff8000000000000ull;  // a NaN all the same
  __hip_atomic_store(reinterpret_cast<unsigned long long *>(slot), b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Householder tridiagonalisation of every matrix of the launch at once.  A column's step is a
// matrix-vector product and a rank-2 update, microseconds of arithmetic at n of a thousand, so the
// cost is what surrounds it: as four launches a column (15 us and the gaps between them, the matrix
// read and written through L2 each time) n = 1237 took 25 ms; now 5.7 ms, 4.65 us a column (5.3 at n = 2047,
// 6.3 at 2400), of which the exchange's way through the Infinity Cache is most.  Here
//   - the matrix lives in registers: workgroup g of the matrix's G holds rows g, g + G, ..., thread t of
//     it the columns t + e * (its threads), so a step touches no memory but the exchange, and a
//     thread's share of the vectors v, w and of row k is as small as its share of a row;
//   - every workgroup keeps v and w for itself and computes them in the same order, so that one
//     exchange a step is enough: workgroups publish (A v)_i of their rows and, of row k + 1, its
//     elements before the step's own update, which every workgroup then applies itself;
//   - a published double is its own flag: slots start out as a NaN pattern that no result has
//     (another one is written for it), every step has slots of its own, and readers poll them
//     with relaxed agent-scope loads, so no fence or counter is involved.
// The launch is cooperative: all workgroups are resident, and a poll that outlasts `spins` ends
// its workgroup with *fail set, which ends the others the same way.
template <int NWV, int NE, int R>
__global__ __launch_bounds__(64 * NWV, NWV / 4) void k_tridiag(const TriProb *probs, const int *wg_prob, int *fail,
                                                                   int spins) {
  constexpr int NT = 64 * NWV;
  __shared__ double lv[2][NT * NE];  // v of the last two steps (a row's own element)
  __shared__ double part[NWV][R];    // per wave: the rows' parts of A v
  __shared__ double pi[R];           // (A v)_i of this workgroup's rows
  __shared__ double red1[NWV], red2[NWV], sc[3];
  __shared__ int failed;
  const TriProb P = probs[wg_prob[blockIdx.x]];
  const int n = P.n, tid = threadIdx.x, lane = tid & 63, G = P.G;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = static_cast<int>(blockIdx.x) - P.wg0;
  double a[R][NE], x[NE], v[NE], w[NE];
  if (tid == 0) failed = 0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int i = r * G + g;
#pragma unroll
    for (int e = 0; e < NE; ++e) a[r][e] = (i < n && tid + NT * e < n) ? P.A[i * P.lda + tid + NT * e] : 0.0;
  }
#pragma unroll
  for (int e = 0; e < NE; ++e) {
    x[e] = tid + NT * e < n ? P.A[tid + NT * e] : 0.0;  // row 0
    v[e] = 0.0;
    w[e] = 0.0;
  }
  // sum over the workgroup of one value per thread, in wave order (the caller's barrier between)
  auto total = [&](const double *red) {
    double t = red[0];
#pragma unroll
    for (int q = 1; q < NWV; ++q) t += red[q];
    return t;
  };
  double bprev = 0.0, hprev = 0.0;  // the last step's beta and beta (p . v) / 2
  for (int k = 0; k < n - 2; ++k) {
    const int par = k & 1;
    // reflector of row k: x = A[k][k+1..], v = x - alpha e1, beta = 2 / v^T v
    double s = 0.0;
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      const int j = tid + NT * e;
      if (j > k + 1) s += x[e] * x[e];  // zero past n
      if (j == k) sc[0] = x[e];
      if (j == k + 1) sc[1] = x[e];
    }
    s = wave_sum_last(s);
    if (lane == 63) red1[wave] = s;
    __syncthreads();
    s = total(red1);
    const double x0 = sc[1];
    double beta = 0.0, alpha = x0, v0 = 0.0;
    if (s > 0.0) {
      const double mu = sqrt(x0 * x0 + s);
      alpha = (x0 >= 0.0) ? -mu : mu;
      v0 = x0 - alpha;
      beta = 2.0 / (v0 * v0 + s);
    }
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      const int j = tid + NT * e;
      x[e] = (j > k + 1 && beta != 0.0) ? x[e] : (j == k + 1 ? v0 : 0.0);  // now the new v
      lv[par][j] = x[e];
    }
    if (g == k % G) {
#pragma unroll
      for (int e = 0; e < NE; ++e)
        if (tid + NT * e < n) P.V[static_cast<int64_t>(k) * n + tid + NT * e] = x[e];
      if (tid == 0) {
        P.beta[k] = beta;
        P.d[k] = sc[0];
        P.e[k] = alpha;
      }
    }
    // own rows: the pending update, then their part of A v
    double *xp = P.X + static_cast<int64_t>(k) * 2 * n, *xr = xp + n;
    double raw[NE];
#pragma unroll
    for (int e = 0; e < NE; ++e) raw[e] = 0.0;
#pragma unroll
    for (int q = 0; q < R; q += 4) {
      if ((q + 3) * G + g <= k || q * G + g >= n) continue;  // no live row in these four
      double acc[4];
#pragma unroll
      for (int r = q; r < q + 4; ++r) {
        const int i = r * G + g;
        acc[r - q] = 0.0;
        if (i > k && i < n) {
          double vi = 0.0, wi = 0.0;
          if (k > 0) {
            vi = lv[par ^ 1][i];
            wi = bprev * pi[r] - hprev * vi;
          }
#pragma unroll
          for (int e = 0; e < NE; ++e) {
            a[r][e] -= vi * w[e] + wi * v[e];
            acc[r - q] += a[r][e] * x[e];
          }
          if (i == k + 1) {
#pragma unroll
            for (int e = 0; e < NE; ++e) {
              const int j = tid + NT * e;
              raw[e] = a[r][e];
              if (G > 1 && j > k && j < n) publish(xr + j, a[r][e]);
            }
          }
        }
      }
      const double t = wave_sum_4(acc);
      if ((lane & 15) == 0) part[wave][q + packed_row(lane >> 4)] = t;
    }
    __syncthreads();
    if (tid < R) {
      const int i = tid * G + g;
      if (i > k && i < n) {
        double t = part[0][tid];
#pragma unroll
        for (int q = 1; q < NWV; ++q) t += part[q][tid];
        pi[tid] = t;
        if (G > 1) publish(xp + i, t);
      }
    }
    double p[NE];
    if (G == 1) {
      __syncthreads();
#pragma unroll
      for (int e = 0; e < NE; ++e) {
        const int j = tid + NT * e;
        p[e] = (j > k && j < n) ? pi[min(j, R - 1)] : 0.0;  // row j is slot j
      }
    } else {
      unsigned todo = 0;
#pragma unroll
      for (int e = 0; e < NE; ++e) {
        const int j = tid + NT * e;
        p[e] = raw[e] = 0.0;
        if (j > k && j < n) todo |= 3u << (2 * e);
      }
      for (int spin = 0; todo != 0; ++spin) {
        unsigned long long pv[NE], rv[NE];
#pragma unroll
        for (int e = 0; e < NE; ++e) {
          const int j = tid + NT * e;
          pv[e] = rv[e] = kEmpty;
          if (todo >> (2 * e) & 1)
            pv[e] = __hip_atomic_load(reinterpret_cast<unsigned long long *>(xp + j), __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_AGENT);
          if (todo >> (2 * e) & 2)
            rv[e] = __hip_atomic_load(reinterpret_cast<unsigned long long *>(xr + j), __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_AGENT);
        }
#pragma unroll
        for (int e = 0; e < NE; ++e) {
          if (pv[e] != kEmpty) {
            p[e] = __longlong_as_double(pv[e]);
            todo &= ~(1u << (2 * e));
          }
          if (rv[e] != kEmpty) {
            raw[e] = __longlong_as_double(rv[e]);
            todo &= ~(2u << (2 * e));
          }
        }
        if (spin >= spins) {
          failed = 1;
          break;
        }
      }
    }
    // w = p - (beta p^T v / 2) v with p = beta A v (beta first: A v is of the matrix' scale squared, and its
    // product with v would leave the range past 1e+-103); then row k + 1 as this step leaves it
    double pv = 0.0;
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      p[e] *= beta;
      pv += p[e] * x[e];
      if (tid + NT * e == k + 1) sc[2] = p[e];
    }
    pv = wave_sum_last(pv);
    if (lane == 63) red2[wave] = pv;
    __syncthreads();
    if (failed) {
      if (tid == 0) *fail = 1;
      return;
    }
    hprev = 0.5 * beta * total(red2);
    bprev = beta;
    const double wk1 = sc[2] - hprev * v0;
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      const int j = tid + NT * e;
      v[e] = x[e];
      w[e] = p[e] - hprev * x[e];
      x[e] = (j > k && j < n) ? raw[e] - (v0 * w[e] + wk1 * v[e]) : 0.0;
    }
  }
  // the last 2 x 2 block: row n - 2 is x, the last diagonal element its owner's
#pragma unroll
  for (int e = 0; e < NE; ++e) {
    const int j = tid + NT * e;
    if (g == 0 && n >= 2 && j == n - 2) P.d[j] = x[e];
    if (g == 0 && n >= 2 && j == n - 1) P.e[n - 2] = x[e];
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (j == n - 1 && r * G + g == n - 1) {
        double vi = 0.0, wi = 0.0;
        if (n > 2) {
          vi = lv[(n - 3) & 1][n - 1];
          wi = bprev * pi[r] - hprev * vi;
        }
        P.d[n - 1] = a[r][e] - (vi * w[e] + wi * v[e]);
      }
  }
}

__global__ void k_fill_empty(unsigned long long *p, int64_t n) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) p[i] = kEmpty;
}

typedef double v4d __attribute__((ext_vector_type(4)));
typedef double v2du __attribute__((ext_vector_type(2), aligned(8)));  // two doubles of a row of any stride

// T of each compact-WY block of kWY reflectors, k0 = items[].at: H_k0 ... H_(k0+kb-1) = I - V^T T V
// with T_jj = beta_j and T[0:j, j] = -beta_j T[0:j, 0:j] G[0:j, j], G the Gram matrix of the block's
// rows of V.  G's ten 16 x 16 tiles on or above the diagonal on the FP64 matrix cores: each wave
// takes a quarter of the columns, 16 at a time (a lane's four elements of a row are the k of four
// steps, in the same order for both operands), and the parts are added in LDS.
__global__ __launch_bounds__(256) void k_wy_t(const TriProb *probs, const BatchWyItem *items) {
  __shared__ double G[kWY][kWY + 1];
  __shared__ double Ts[kWY][kWY + 1];
  __shared__ double bet[kWY];
  const BatchWyItem it = items[blockIdx.x];
  const TriProb P = probs[it.prob];
  const int n = P.n, tid = threadIdx.x, k0 = it.at, kb = min(kWY, n - 2 - k0);
  const int lane = tid & 63, wave = tid >> 6, li = lane & 15, lq = lane >> 4;
  v4d acc[10];
#pragma unroll
  for (int t = 0; t < 10; ++t) acc[t] = v4d{0.0, 0.0, 0.0, 0.0};
  auto load = [&](double(&v)[4][4], int c0) {
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const double *row = P.V + static_cast<int64_t>(k0 + 16 * g + li) * n + c0 + 4 * lq;
      const bool in = 16 * g + li < kb;
      if (c0 + 16 <= n) {
        const v2du a = in ? *reinterpret_cast<const v2du *>(row) : v2du{0.0, 0.0};
        const v2du b = in ? *reinterpret_cast<const v2du *>(row + 2) : v2du{0.0, 0.0};
        v[g][0] = a[0];
        v[g][1] = a[1];
        v[g][2] = b[0];
        v[g][3] = b[1];
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[g][e] = (in && c0 + 4 * lq + e < n) ? row[e] : 0.0;
      }
    }
  };
  double cur[4][4], nxt[4][4];
  int c0 = ((k0 + 1) / 16 + wave) * 16;  // the block's rows are zero before column k0 + 1
  if (c0 < n) load(cur, c0);
  for (; c0 < n; c0 += 64) {
    if (c0 + 64 < n) load(nxt, c0 + 64);
    int t = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = i; j < 4; ++j, ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(cur[i][e], cur[j][e], acc[t], 0, 0, 0);
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
      for (int e = 0; e < 4; ++e) cur[g][e] = nxt[g][e];
  }
  if (tid < kb) bet[tid] = P.beta[k0 + tid];
  for (int w = 0; w < 4; ++w) {  // the waves' parts in order
    if (wave == w) {
      int t = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = i; j < 4; ++j, ++t)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            double &g = G[16 * i + lq + 4 * e][16 * j + li];
            g = (w == 0 ? 0.0 : g) + acc[t][e];
          }
    }
    __syncthreads();
  }
  for (int j = 0; j < kb; ++j) {
    if (tid < j) {
      double t = 0.0;
      for (int q = tid; q < j; ++q) t += Ts[tid][q] * G[q][j];
      Ts[tid][j] = -bet[j] * t;
    } else if (tid == j) {
      Ts[j][j] = bet[j];
    } else if (tid < kb) {
      Ts[tid][j] = 0.0;
    }
    __syncthreads();
  }
  double *T = P.V + static_cast<int64_t>(n) * n + static_cast<int64_t>(k0 / kWY) * kWY * kWY;
  for (int e = tid; e < kb * kb; e += 256) T[e] = Ts[e / kb][e % kb];
}

// Shapes of k_tridiag: rows of up to 64 nwv ne elements, r of them a workgroup.  Of the two r of a row
// length the smaller gives the shortest step, the larger (as much as the registers hold) room for
// more matrices in a launch.  Past 2048 rows 256 compute units need 12 rows each: at n = 2400 five
// elements a thread of eight waves take 20.6 ms a solve, four of twelve waves 27.2; six of eight
// spill, so twelve waves take the rest.
struct TriShape {
  int nwv, ne, r;
  const void *fn;
};
#define DACP_TRI(nwv, ne, r) {nwv, ne, r, reinterpret_cast<const void *>(k_tridiag<nwv, ne, r>)}
const TriShape kTriShapes[] = {
    DACP_TRI(4, 1, 8), DACP_TRI(4, 1, 64), DACP_TRI(8, 1, 8), DACP_TRI(8, 1, 64), DACP_TRI(12, 1, 8), DACP_TRI(12, 1, 48),
    DACP_TRI(8, 2, 8), DACP_TRI(8, 2, 36), DACP_TRI(8, 3, 8), DACP_TRI(8, 3, 24), DACP_TRI(8, 4, 8), DACP_TRI(8, 4, 16),
    DACP_TRI(8, 5, 12), DACP_TRI(12, 4, 12),
};
#undef DACP_TRI

int tri_wgs(int n, int r) { return (n + r - 1) / r; }

// Z <- Z Q^T for one matrix of more rows than k_wy_apply's registers take, the same product a block
// at a time through the GEMM: W1 = Z V_j^T, W2 = W1 T_j^T, Z -= W2 V_j on the columns after k0.
// w: 2 n kWY doubles.  3.8 ms at n = 2400; one reflector a launch (15 us each) took 36.
dacp_status wy_gemm(dacp_ctx ctx, int n, const double *V, double *Z, double *w) {
  hipStream_t st = ctx->stream;
  const double *T = V + static_cast<int64_t>(n) * n;
  double *w2 = w + static_cast<int64_t>(n) * kWY;
  for (int k0 = (n - 3) / kWY * kWY; k0 >= 0; k0 -= kWY) {
    const int kb = std::min(kWY, n - 2 - k0), c0 = k0 + 1;
    const double *Vj = V + static_cast<int64_t>(k0) * n + c0;
    const double *Tj = T + static_cast<int64_t>(k0 / kWY) * kWY * kWY;
    DACP_HIP(ctx, launch_dgemm(0, 1, n, kb, n - c0, 1.0, Z + c0, n, Vj, n, 0.0, w, kb, 0, st));
    DACP_HIP(ctx, launch_dgemm(0, 1, n, kb, kb, 1.0, w, kb, Tj, kb, 0.0, w2, kb, 0, st));
    DACP_HIP(ctx, launch_dgemm(0, 0, n, n - c0, kb, -1.0, w2, kb, Vj, n, 1.0, Z + c0, n, 0, st));
  }
  return DACP_OK;
}

}  // namespace

bool syev_on_chip(dacp_ctx ctx, int n) {
  int row = 0, wgs = 0;
  for (const TriShape &s : kTriShapes) {
    const int len = 64 * s.nwv * s.ne;
    if (len < n || (row && len > row)) continue;
    row = len;
    wgs = tri_wgs(n, s.r);  // the last shape of a row length has the most rows a workgroup
  }
  return row > 0 && wgs <= ctx->num_cus;
}

// The tridiagonalisations: matrices of similar size go together, largest first, each launch taking
// as many as the compute units hold (one workgroup each).  no_exchange: the runtime refused a cooperative launch
// (it gives them to one process at a time on a device), or an exchange waited too long (other processes'
// kernels hold compute units); the results are not there.
static dacp_status tridiagonalise(dacp_ctx ctx, std::vector<TriProb> &probs, TriProb *dprobs, bool &no_exchange) {
  hipStream_t st = ctx->stream;
  const int np = static_cast<int>(probs.size());
  std::vector<int> order(np);
  std::iota(order.begin(), order.end(), 0);
  std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return probs[a].n > probs[b].n; });
  struct Launch {
    const void *fn;
    int threads, wg0, wgs;
    bool shared;  // some matrix has more than one workgroup
  };
  std::vector<Launch> launches;
  std::vector<int> wg_prob;
  for (int at = 0; at < np;) {
    auto rows = [](const TriShape &s) { return 64 * s.nwv * s.ne; };
    const int row = [&] {
      for (const TriShape &s : kTriShapes)
        if (rows(s) >= probs[order[at]].n) return rows(s);
      return 0;
    }();
    // the smaller R when the rest of the list fits one launch with it, else the larger
    const TriShape *shape = nullptr;
    for (const TriShape &s : kTriShapes) {
      if (rows(s) != row) continue;
      int need = 0;
      for (int q = at; q < np; ++q) need += tri_wgs(probs[order[q]].n, s.r);
      shape = &s;
      if (need <= ctx->num_cus) break;
    }
    if (!shape || tri_wgs(probs[order[at]].n, shape->r) > ctx->num_cus)  // syev_on_chip's rule
      return set_err(ctx, DACP_E_HIP, "eigensolver: matrix does not fit the device's compute units");
    Launch ln{shape->fn, 64 * shape->nwv, static_cast<int>(wg_prob.size()), 0, false};
    for (; at < np; ++at) {
      TriProb &p = probs[order[at]];
      const int g = tri_wgs(p.n, shape->r);
      if (ln.wgs + g > ctx->num_cus) break;
      p.G = g;
      p.wg0 = ln.wgs;
      ln.wgs += g;
      ln.shared = ln.shared || g > 1;
      wg_prob.insert(wg_prob.end(), g, order[at]);
    }
    launches.push_back(ln);
  }
  DevBuf dwg;
  DACP_HIP(ctx, dwg.alloc((wg_prob.size() + 1) * sizeof(int)));
  int *fail = dwg.as<int>() + wg_prob.size();
  wg_prob.push_back(0);
  DACP_TRY(to_device(ctx, dwg.p, wg_prob.data(), wg_prob.size() * sizeof(int)));
  DACP_TRY(to_device(ctx, dprobs, probs.data(), sizeof(TriProb) * np));
  for (const TriProb &p : probs)
    if (p.G > 1) {
      const int64_t nx = 2 * static_cast<int64_t>(p.n) * p.n;
      hipLaunchKernelGGL(k_fill_empty, dim3(static_cast<unsigned>((nx + 255) / 256)), dim3(256), 0, st,
                         reinterpret_cast<unsigned long long *>(p.X), nx);
    }
  DACP_HIP(ctx, hipGetLastError());
  bool refused = false;
  for (const Launch &ln : launches) {
    const TriProb *ap = dprobs;
    const int *aw = dwg.as<int>() + ln.wg0;
    int spins = ctx->tri_spins;
    void *args[] = {&ap, &aw, &fail, &spins};
    // matrices of one workgroup exchange nothing: an ordinary launch (eigenvalues of 5 rows: 135 us, as a
    // cooperative one 153, and a process without one waits about 1 us less at each synchronisation)
    if (ln.shared) {
      if (hipLaunchCooperativeKernel(ln.fn, dim3(ln.wgs), dim3(ln.threads), args, 0, st) != hipSuccess) {
        const hipError_t e = hipGetLastError();
        vlog("eigensolver: cooperative launch refused: %s", hipGetErrorString(e));
        refused = true;
        break;
      }
    } else {
      DACP_HIP(ctx, hipLaunchKernel(ln.fn, dim3(ln.wgs), dim3(ln.threads), args, 0, st));
    }
  }
  int failed = 0;
  DACP_TRY(to_host(ctx, &failed, fail, sizeof(int)));
  no_exchange = refused || failed != 0;
  return DACP_OK;
}

// One round: np matrices together.  A is only read, so a round that fails can be run again, and one without an
// exchange is left to the caller.
static dacp_status solve_round(dacp_ctx ctx, const SyevJob *jobs, int np, bool &no_exchange) {
  hipStream_t st = ctx->stream;
  size_t zs = 0, vs = 0, xs = 0, ds = 0;
  for (int i = 0; i < np; ++i) {
    const size_t n = jobs[i].n, nn = n * n;
    if (!jobs[i].Z) zs += nn;
    vs += batch_syev_work_doubles(jobs[i].n);
    xs += std::max(dc_work_doubles(jobs[i].n), 2 * nn);
    ds += 3 * n;
  }
  DevBuf bz, bv, bx, bd, bp, bi;
  if (zs) DACP_HIP(ctx, bz.alloc(zs * sizeof(double)));
  DACP_HIP(ctx, bv.alloc(vs * sizeof(double)));
  DACP_HIP(ctx, bx.alloc(xs * sizeof(double)));  // the exchange, then the divide and conquer's scratch
  DACP_HIP(ctx, bd.alloc(ds * sizeof(double)));
  DACP_HIP(ctx, bp.alloc(sizeof(TriProb) * np));
  double *z = bz.as<double>(), *v = bv.as<double>(), *x = bx.as<double>(), *d = bd.as<double>();
  std::vector<TriProb> probs(np);
  std::vector<DcJob> dc(np);
  std::vector<BatchWyItem> prep, apply;
  std::vector<BatchEigProblem> wy(np);
  int max_n = 0;
  for (int i = 0; i < np; ++i) {
    const SyevJob &j = jobs[i];
    const size_t nn = static_cast<size_t>(j.n) * j.n;
    probs[i] = {j.A, j.lda, v, x, d, d + j.n, d + 2 * j.n, j.n, 1, 0};
    dc[i] = {j.n, d, d + j.n, j.Z ? j.Z : z, x, j.w};
    wy[i] = {nullptr, dc[i].Z, v, nullptr, nullptr, j.n};
    if (!j.Z) z += nn;
    v += batch_syev_work_doubles(j.n);
    x += std::max(dc_work_doubles(j.n), 2 * nn);
    d += 3 * static_cast<size_t>(j.n);
    if (j.Z && j.n > 2) {
      if (j.n <= kWyApplyMaxN) max_n = std::max(max_n, j.n);
      for (int k0 = 0; k0 < j.n - 2; k0 += kWY) prep.push_back({i, k0});
      if (j.n <= kWyApplyMaxN)
        for (int r0 = 0; r0 < j.n; r0 += kWyRows) apply.push_back({i, r0});
    }
  }
  no_exchange = false;
  DACP_TRY(tridiagonalise(ctx, probs, bp.as<TriProb>(), no_exchange));
  if (no_exchange) return DACP_OK;
  DACP_TRY(dc_tridiag_jobs(ctx, dc));
  if (!prep.empty()) {
    DevBuf bw;
    const size_t np_items = prep.size();
    prep.insert(prep.end(), apply.begin(), apply.end());
    DACP_HIP(ctx, bi.alloc(prep.size() * sizeof(BatchWyItem)));
    DACP_HIP(ctx, bw.alloc(wy.size() * sizeof(BatchEigProblem)));
    DACP_TRY(to_device(ctx, bi.p, prep.data(), prep.size() * sizeof(BatchWyItem)));
    DACP_TRY(to_device(ctx, bw.p, wy.data(), wy.size() * sizeof(BatchEigProblem)));
    hipLaunchKernelGGL(k_wy_t, dim3(static_cast<unsigned>(np_items)), dim3(256), 0, st, bp.as<TriProb>(),
                       bi.as<BatchWyItem>());
    DACP_HIP(ctx, hipGetLastError());
    DACP_HIP(ctx, launch_wy_apply(bw.as<BatchEigProblem>(), bi.as<BatchWyItem>() + np_items,
                                  static_cast<int>(apply.size()), max_n, st));
    for (int i = 0; i < np; ++i)  // the divide and conquer's scratch is free again
      if (jobs[i].Z && jobs[i].n > kWyApplyMaxN)
        DACP_TRY(wy_gemm(ctx, jobs[i].n, wy[i].work, jobs[i].Z, probs[i].X));
    DACP_HIP(ctx, hipStreamSynchronize(st));  // the scratch is released on return
  }
  return DACP_OK;
}

// The matrices of a round without an exchange, in memory: one after the other column by column (about 20 us a row:
// 4.0 ms at 200 rows, 13.9 at 664), or, where that takes longer, together with a workgroup each (about 0.3 us times
// the square of the largest's rows: 32 of 200 rows 14 ms, 8 of 664 rows 127).
static dacp_status solve_apart(dacp_ctx ctx, const SyevJob *jobs, int np) {
  std::vector<int> n;
  std::vector<double *> A, w, Z;
  int64_t rows = 0, max_n = 0;
  bool whole = true;
  for (int i = 0; i < np; ++i) {
    n.push_back(jobs[i].n);
    A.push_back(jobs[i].A);
    w.push_back(jobs[i].w);
    Z.push_back(jobs[i].Z);
    rows += jobs[i].n;
    max_n = std::max<int64_t>(max_n, jobs[i].n);
    whole = whole && jobs[i].lda == jobs[i].n;
  }
  if (whole && np > 1 && max_n <= kBatchEigMaxN && 60 * rows > max_n * max_n)
    return batch_syev_each(ctx, np, n.data(), A.data(), w.data(), Z.data());
  for (int i = 0; i < np; ++i) DACP_TRY(gpu_syev(ctx, jobs[i].n, jobs[i].A, jobs[i].lda, jobs[i].w, jobs[i].Z, false));
  return DACP_OK;
}

static dacp_status solve_jobs(dacp_ctx ctx, const std::vector<SyevJob> &all) {
  std::vector<SyevJob> jobs;
  for (const SyevJob &j : all) {
    if (syev_on_chip(ctx, j.n)) jobs.push_back(j);
    else DACP_TRY(gpu_syev(ctx, j.n, j.A, j.lda, j.w, j.Z));
  }
  // the whole list, or, where the device has not that much scratch (4 n^2 doubles a matrix, 5 without
  // Z) left, half as many at a time until it has
  int per = static_cast<int>(jobs.size());
  for (int at = 0, np = per; at < np;) {
    const int take = std::min(per, np - at);
    bool no_exchange = false;
    dacp_status st = solve_round(ctx, jobs.data() + at, take, no_exchange);
    if (st == DACP_OK && no_exchange) {
      vlog("eigensolver: no exchange between compute units, %d matrices in memory", take);
      DACP_TRY(solve_apart(ctx, jobs.data() + at, take));  // destroys A: a failure is not tried again
    }
    if (st == DACP_E_NOMEM && take > 1) {
      (void)hipGetLastError();
      ctx->err.clear();
      per = (take + 1) / 2;
    } else if (st != DACP_OK) {
      return st;
    } else {
      at += take;
    }
  }
  return DACP_OK;
}

dacp_status syev_jobs(dacp_ctx ctx, const std::vector<SyevJob> &jobs) {
  try {
    return solve_jobs(ctx, jobs);
  } catch (...) {  // the host tables; the callers are C entry points
    return set_err(ctx, DACP_E_NOMEM, "eigensolver: host allocation failed");
  }
}

}  // namespace dacp
