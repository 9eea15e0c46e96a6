// Batched Chebyshev path for many small realisations (L <= 14) in one persistent launch.
//
// Workgroup g owns column j of realisation r (descriptor cols[g]) and runs that column's
// whole recurrence on-chip: the recurrence terms in registers (2^L / 512 elements per thread) and
// the vector being applied also in LDS (one 2^L-long column, <= 128 KB in FP64).  In order it runs
//   1. the exp-semicircle filter T_K(F) psi (Sec. II.A, Eqs. F, filter) with the damped
//      recurrence T^_{k+1} = alpha H(H T^_k) + beta T^_k + gamma T^_{k-1}: the first K - tail
//      orders in FP32 (FP32 storage and accumulation), the last `tail` orders in FP64;
//   2. column normalisation (a fixed-order workgroup reduction);
//   3. the Chebyshev evolution T_{k+1} = 2 G T_k - T_{k-1}, G = H / E_b (Sec. II.B), storing
//      the panels T_{k_m - 1}, T_{k_m} into the realisation's basis V (App. C, Eq. set2) and
//      checking |T_{k_m}| <= |psi_E| at every sample.
// A call's columns of a basis can also run part 1 or part 3 alone (BatchCol::mode).
//
// What bounds an apply is the reads of its flips: a column of 2^14 read from LDS once per single-spin
// flip is 14 x 128 KB at 128 bytes a cycle, 6 us of a measured 10.  So the index bits are dealt
// s = lane + 64 wave + 512 i: bits 9.. pick one of the thread's own registers, bits 0-3 are DPP
// moves of the vector unit, and only bits 4-8 read LDS; each term costs its multiply-add and, by
// bit, nothing, two to four moves, or one LDS read.  Those terms come as one coefficient per bit
// (xc); every other flip (two spins, or a sign) reads LDS through the flip table.  Two terms of
// 2^14 doubles take 64 registers each with 512 threads a workgroup, so none lives in memory.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "internal.h"
#include "wave.h"

namespace dacp {

namespace {

constexpr int kBT = 512;  // threads per workgroup
constexpr int kBW = kBT / 64;

typedef const __attribute__((address_space(4))) BatchCol *ConstBatchCols;
typedef const __attribute__((address_space(4))) FlipEntry *ConstFlipTable;
typedef const __attribute__((address_space(4))) int *ConstInts;
typedef const __attribute__((address_space(4))) double *ConstDoubles;

// The off-diagonal part of one realisation's H.
struct OffDiag {
  ConstDoubles xc;         // coefficient of sigma^x_b, b < 14 (0 where there is none)
  ConstFlipTable flips;    // every other flip, sign-free ones first
  int nplain, nflip;
};

// threadIdx.x * scale, opaque to loop-invariant code motion: an empty asm statement (no
// instruction) redefines the value, so the addresses derived from it are formed where they are
// used instead of being hoisted out of the step loops and held in registers for the whole kernel.
// Global accesses are a uniform base plus a 32-bit byte offset (every offset here is < 2^32,
// checked on the host), so the per-element address is one 32-bit register.
__device__ __forceinline__ uint32_t tid_off(uint32_t scale) {
  uint32_t o = threadIdx.x * scale;
  asm volatile("" : "+v"(o));
  return o;
}

template <typename T>
__device__ __forceinline__ T ld_at(const T *base, uint32_t byte_off) {
  return *reinterpret_cast<const T *>(reinterpret_cast<const char *>(base) + byte_off);
}
template <typename T>
__device__ __forceinline__ void st_at(T *base, uint32_t byte_off, T x) {
  *reinterpret_cast<T *>(reinterpret_cast<char *>(base) + byte_off) = x;
}

// x is formed here: left alone, the compiler moves every chunk's last operations behind the last
// chunk's, and their inputs then outnumber the registers.
template <typename T>
__device__ __forceinline__ void set_now(T &x, T v) {
  x = v;
  asm volatile("" : "+v"(x));
}

template <int kCtrl>
__device__ __forceinline__ double dpp(double v) {
  return dpp_move<kCtrl, 0xf>(v);
}
template <int kCtrl>
__device__ __forceinline__ float dpp(float v) {
  return __int_as_float(dpp_move<kCtrl, 0xf>(__float_as_int(v)));
}
// The value of lane (lane ^ 2^B), B < 4.
template <int B, typename T>
__device__ __forceinline__ T lane_flip(T v) {
  if constexpr (B == 0) return dpp<0xB1>(v);             // quad_perm 1 0 3 2
  else if constexpr (B == 1) return dpp<0x4E>(v);        // quad_perm 2 3 0 1
  else if constexpr (B == 2) return dpp<0x1B>(dpp<0x141>(v));  // row_half_mirror, quad_perm 3 2 1 0
  else return dpp<0x128>(v);                             // row_ror 8
}

// v with the sign bit of `bit31` applied.
__device__ __forceinline__ double sign_xor(double v, uint32_t bit31) {
  return __hiloint2double(__double2hiint(v) ^ static_cast<int>(bit31), __double2loint(v));
}
__device__ __forceinline__ float sign_xor(float v, uint32_t bit31) {
  return __int_as_float(__float_as_int(v) ^ static_cast<int>(bit31));
}

// The flip table's terms of the thread's elements ib .. ib + C - 1.  The source of element tid + 512 i under
// mask x is (tid ^ x's low 9 bits) + ((512 i) ^ the others): one lane offset a flip and a uniform part an
// element.  A sign is the parity of the source under the z-mask, which is linear: the lane's part and the
// mask's go to the coefficient, and what is left for an element is the parity of i's low three bits under
// bits 9 to 11 of the z-mask.  The next flip's entry is loaded under this one's reads (the table ends
// with a spare one): a flip's time is the instructions it issues and the latency of one read, not the
// reads' bandwidth (0.43 us at 2^14 rows in FP64).  With the entry waited for and an index and a sign
// formed per element it took 0.75 us, 1.3 with a sign; now 0.50 and 0.85.
template <typename T, int C>
__device__ __forceinline__ void table_flips(T (&s)[C], const T *lds, const OffDiag &od, int ib) {
  constexpr uint32_t kLane = kBT - 1, kSh = sizeof(T) == 8 ? 3 : 2;
  const char *ldsb = reinterpret_cast<const char *>(lds);
  ConstFlipTable next = od.flips;
  uint32_t xm = next->xmask, zm = next->zmask;
  double cf = next->coef;
  auto flip = [&](auto sgn) {
    constexpr bool kSigned = decltype(sgn)::value;
    const uint32_t xh = xm & ~kLane, xl = tid_off(1u) ^ (xm & kLane), zt = zm;
    T c = static_cast<T>(cf);
    if constexpr (kSigned)
      c = sign_xor(c, static_cast<uint32_t>(__popc(xl & zt & kLane) + __popc((xh ^ static_cast<uint32_t>(ib * kBT)) & zt & ~kLane))
                          << 31);
    T g[C];
#pragma unroll
    for (int i = 0; i < C; ++i)
      g[i] = *reinterpret_cast<const T *>(ldsb + ((xl << kSh) + (static_cast<uint32_t>((ib + i) * kBT) << kSh ^ xh << kSh)));
    ++next;
    xm = next->xmask;
    zm = next->zmask;
    cf = next->coef;
#pragma unroll
    for (int i = 0; i < C; ++i) {
      if constexpr (kSigned)
        g[i] = sign_xor(g[i], (i & 1 ? zt << 22 & 1u << 31 : 0u) ^ (i & 2 ? zt << 21 & 1u << 31 : 0u) ^
                                  (i & 4 ? zt << 20 & 1u << 31 : 0u));
      s[i] += c * g[i];
    }
  };
#pragma nounroll
  for (int t = 0; t < od.nplain; ++t) flip(std::false_type());
#pragma nounroll
  for (int t = od.nplain; t < od.nflip; ++t) flip(std::true_type());
}

// s[i] = (H v) of the thread's elements ib .. ib + C - 1; lds holds v (elements past 2^L zero).
// Elements go in chunks of at most 8, which bounds the loads in flight; a chunk's diagonal entries
// are loaded first and applied last, so their latency runs under the flips.
template <typename T, int E, int C, bool kSingle>
__device__ __forceinline__ void chunk_apply(T (&s)[C], const T (&v)[E], const T *lds, const T *diag, const OffDiag &od,
                                            uint32_t D, int ib) {
  T dg[C];
#pragma unroll
  for (int i = 0; i < C; ++i) {
    const uint32_t o = E == 1 ? min(tid_off(1u), D - 1) * sizeof(T) : tid_off(sizeof(T));
    dg[i] = ld_at(diag, o + static_cast<uint32_t>((ib + i) * kBT * sizeof(T)));
  }
#pragma unroll
  for (int i = 0; i < C; ++i) s[i] = T(0);
  if constexpr (kSingle) {
#pragma unroll
    for (int b = 4; b < 9; ++b) {
      const T c = static_cast<T>(od.xc[b]);
      const T *src = lds + (tid_off(1u) ^ (1u << b)) + ib * kBT;
#pragma unroll
      for (int i = 0; i < C; ++i) s[i] += c * src[i * kBT];
    }
    const T c0 = static_cast<T>(od.xc[0]), c1 = static_cast<T>(od.xc[1]), c2 = static_cast<T>(od.xc[2]),
            c3 = static_cast<T>(od.xc[3]);
#pragma unroll
    for (int i = 0; i < C; ++i) s[i] += c0 * lane_flip<0>(v[ib + i]);
#pragma unroll
    for (int i = 0; i < C; ++i) s[i] += c1 * lane_flip<1>(v[ib + i]);
#pragma unroll
    for (int i = 0; i < C; ++i) s[i] += c2 * lane_flip<2>(v[ib + i]);
#pragma unroll
    for (int i = 0; i < C; ++i) s[i] += c3 * lane_flip<3>(v[ib + i]);
#pragma unroll
    for (int b = 9; (1 << (b - 9)) < E; ++b) {
      const T c = static_cast<T>(od.xc[b]);
#pragma unroll
      for (int i = 0; i < C; ++i) s[i] += c * v[(ib + i) ^ (1 << (b - 9))];
    }
  }
  if (od.nflip > 0) table_flips<T, C>(s, lds, od, ib);
#pragma unroll
  for (int i = 0; i < C; ++i) s[i] += dg[i] * v[ib + i];
}

// out(i, (H v)_i) for every element of this thread: v goes to LDS (between barriers: the previous
// apply's readers are done, then the writers), then chunk by chunk.
template <bool kSingle, typename T, int E, typename Out>
__device__ __forceinline__ void apply(const T (&v)[E], T *lds, const T *diag, const OffDiag &od, uint32_t D, Out out) {
  __syncthreads();
#pragma unroll
  for (int h = 0; h < E; h += 8) {  // LDS offsets reach 64 KB from one address register
    T *dst = lds + tid_off(1u) + h * kBT;
#pragma unroll
    for (int i = h; i < h + 8 && i < E; ++i) dst[(i - h) * kBT] = v[i];
  }
  __syncthreads();
  constexpr int C = E < 8 ? E : 8;
#pragma unroll
  for (int ib = 0; ib < E; ib += C) {
    T s[C];
    asm volatile("" ::: "memory");  // the next chunk's loads stay behind
    chunk_apply<T, E, C, kSingle>(s, v, lds, diag, od, D, ib);
#pragma unroll
    for (int i = 0; i < C; ++i) out(ib + i, s[i]);
  }
}

// Sum over the workgroup in a fixed order, the same value in every thread.
__device__ __forceinline__ double block_sum(double v, double *red) {
  v = wave_sum_last(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 63) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double t = 0.0;
  for (int w = 0; w < kBW; ++w) t += red[w];
  return t;
}

template <int E>
__device__ __forceinline__ double dot(const double (&x)[E], const double (&y)[E], double *red) {
  double p = 0.0;
#pragma unroll
  for (int i = 0; i < E; ++i) p += x[i] * y[i];
  return block_sum(p, red);
}

template <int E>
__device__ __forceinline__ void store_panel(double *V, int64_t ldv, int64_t col, const double (&v)[E], uint32_t D) {
#pragma unroll
  for (int i = 0; i < E; ++i) {
    const uint32_t s = tid_off(1u) + static_cast<uint32_t>(i * kBT);
    if (E > 1 || s < D) st_at(V, (s * static_cast<uint32_t>(ldv) + static_cast<uint32_t>(col)) * 8u, v[i]);
  }
}

template <int E>
__device__ __forceinline__ void swap_arrays(double (&x)[E], double (&y)[E]) {
#pragma unroll
  for (int i = 0; i < E; ++i) {
    const double t = x[i];
    x[i] = y[i];
    y[i] = t;
  }
}

// Store T_kk when kk is a sample order; at k_m also check |T_{k_m}|^2 <= |psi_E|^2 = norm2.
template <int E>
__device__ __forceinline__ void sample_at(const BatchCol &c, ConstInts ks, int &next, int64_t kk, const double (&T)[E],
                                          uint32_t D, double norm2, double *red) {
  if (next >= c.n_samples) return;
  const int64_t km = ks[next];
  if (kk == km - 1) store_panel<E>(c.V, c.ldv, static_cast<int64_t>(2 * next + 1) * c.b, T, D);
  if (kk == km) {
    store_panel<E>(c.V, c.ldv, static_cast<int64_t>(2 * next + 2) * c.b, T, D);
    const double n2 = dot<E>(T, T, red);
    if (!(n2 <= norm2 * (1.0 + 2e-6)) && threadIdx.x == 0)
      atomicMin(c.bound_flag, 2 * next + (isfinite(n2) ? 0 : 1));  // the earliest sample's
    ++next;
  }
}

// Store T_kk into the anchor slot when kk is the next anchor order (the moment projection).
template <int E>
__device__ __forceinline__ void anchor_at(const BatchCol &c, ConstInts ka, int &next, int64_t kk, const double (&T)[E],
                                          uint32_t D) {
  if (next >= c.n_anchor || ka[next] != kk) return;
  store_panel<E>(c.A, c.lda, static_cast<int64_t>(next) * c.b, T, D);
  ++next;
}

// The filter's recurrence from psi in v: on exit v = T^_K and A = T^_(K-1), T^_0 = psi.  Orders run in
// pairs with the two terms' roles swapped, so that no copies are made.
template <bool kSingle, typename T, int E>
__device__ __forceinline__ void filter_first(T (&A)[E], T (&B)[E], T *lds, const T *diag, const OffDiag &od, uint32_t D,
                                             T fa, T fb) {
  T w[E];
  apply<kSingle, T, E>(A, lds, diag, od, D, [&](int i, T x) { set_now(w[i], x); });
  apply<kSingle, T, E>(w, lds, diag, od, D, [&](int i, T x) { set_now(B[i], fa * x + fb * A[i]); });
}
// A <- alpha H (H B) + beta B + gamma A
template <bool kSingle, typename T, int E>
__device__ __forceinline__ void filter_order(T (&A)[E], const T (&B)[E], T *lds, const T *diag, const OffDiag &od,
                                             uint32_t D, T alpha, T beta, T gamma) {
  T w[E];
  apply<kSingle, T, E>(B, lds, diag, od, D, [&](int i, T x) { set_now(w[i], x); });
  apply<kSingle, T, E>(w, lds, diag, od, D, [&](int i, T x) { set_now(A[i], alpha * x + beta * B[i] + gamma * A[i]); });
}
// `count` orders from (A, B) = (T^_(k-1), T^_k); the newest ends in B when count is even, in A when odd.
template <bool kSingle, typename T, int E>
__device__ __forceinline__ void filter_orders(T (&A)[E], T (&B)[E], T *lds, const T *diag, const OffDiag &od, uint32_t D,
                                              T alpha, T beta, T gamma, int count) {
  int k = 0;
  for (; k + 2 <= count; k += 2) {
    filter_order<kSingle, T, E>(A, B, lds, diag, od, D, alpha, beta, gamma);
    filter_order<kSingle, T, E>(B, A, lds, diag, od, D, alpha, beta, gamma);
  }
  if (k < count) filter_order<kSingle, T, E>(A, B, lds, diag, od, D, alpha, beta, gamma);
}

template <int E, bool kSingle>
__device__ __forceinline__ void run_column(const BatchCol &c, const OffDiag &od, ConstInts ks, ConstInts ka,
                                           unsigned char *smem, double *red) {
  const uint32_t D = 1u << c.L;
  double *lds64 = reinterpret_cast<double *>(smem);
  float *lds32 = reinterpret_cast<float *>(smem);
  const bool active = E > 1 || threadIdx.x < D;
  double A[E], v[E];  // T_(k-1), T_k
#pragma unroll
  for (int i = 0; i < E; ++i) {
    const uint32_t s = threadIdx.x + i * kBT;
    v[i] = active ? ld_at(c.psi0, s * static_cast<uint32_t>(c.ld_psi) * 8u) : 0.0;  // start column
    A[i] = v[i];
  }

  if (c.mode != kBatchEvolve) {
    // ---- filter: on exit v = T^_K, A = T^_(K-1)
    int tail = 0;
    if (c.K > 0 && c.n32 >= 1) {
      float Af[E], Bf[E];
#pragma unroll
      for (int i = 0; i < E; ++i) Af[i] = static_cast<float>(v[i]);
      filter_first<kSingle, float, E>(Af, Bf, lds32, c.d32, od, D, static_cast<float>(c.f_first_a),
                             static_cast<float>(c.f_first_b));
      filter_orders<kSingle, float, E>(Af, Bf, lds32, c.d32, od, D, static_cast<float>(c.f_alpha),
                              static_cast<float>(c.f_beta), static_cast<float>(c.f_gamma), c.n32 - 1);
      const bool odd = (c.n32 - 1) & 1;
#pragma unroll
      for (int i = 0; i < E; ++i) {
        v[i] = static_cast<double>(odd ? Af[i] : Bf[i]);
        A[i] = static_cast<double>(odd ? Bf[i] : Af[i]);
      }
      tail = c.K - c.n32;
    } else if (c.K > 0) {
      filter_first<kSingle, double, E>(A, v, lds64, c.d64, od, D, c.f_first_a, c.f_first_b);
      tail = c.K - 1;
    }
    filter_orders<kSingle, double, E>(A, v, lds64, c.d64, od, D, c.f_alpha, c.f_beta, c.f_gamma, tail);
    if (tail & 1) swap_arrays<E>(A, v);
    if (c.mode == kBatchFilter) {  // not normalised: the caller checks the norms
      store_panel<E>(c.V, c.ldv, 0, v, D);
      return;
    }
    // ---- normalise: psi_E = v / |v|
    const double inv = 1.0 / sqrt(dot<E>(v, v, red));
#pragma unroll
    for (int i = 0; i < E; ++i) v[i] *= inv;
  }
  const double norm2 = c.mode == kBatchEvolve ? dot<E>(v, v, red) : 1.0;

  // ---- evolution: A = T_(k-1), v = T_k
  store_panel<E>(c.V, c.ldv, 0, v, D);
  int next = 0, next_a = 0;
  anchor_at<E>(c, ka, next_a, 0, v, D);
#pragma unroll
  for (int i = 0; i < E; ++i) A[i] = v[i];
  apply<kSingle, double, E>(A, lds64, c.d64, od, D, [&](int i, double x) { set_now(v[i], c.inv_e * x); });
  sample_at<E>(c, ks, next, 1, v, D, norm2, red);
  anchor_at<E>(c, ka, next_a, 1, v, D);
  int64_t kmax = c.n_samples > 0 ? ks[c.n_samples - 1] : 1;
  if (c.n_anchor > 0 && ka[c.n_anchor - 1] > kmax) kmax = ka[c.n_anchor - 1];
  const double two_inv_e = 2.0 * c.inv_e;
  for (int64_t k = 1; k < kmax; k += 2) {
    apply<kSingle, double, E>(v, lds64, c.d64, od, D, [&](int i, double x) { set_now(A[i], two_inv_e * x - A[i]); });
    sample_at<E>(c, ks, next, k + 1, A, D, norm2, red);
    anchor_at<E>(c, ka, next_a, k + 1, A, D);
    if (k + 1 >= kmax) break;
    apply<kSingle, double, E>(A, lds64, c.d64, od, D, [&](int i, double x) { set_now(v[i], two_inv_e * x - v[i]); });
    sample_at<E>(c, ks, next, k + 2, v, D, norm2, red);
    anchor_at<E>(c, ka, next_a, k + 2, v, D);
  }
}

// Elements per thread: 2^L / 512, at least 1.  Without single-spin terms (kSingle false) their sweeps are
// not there at all; a branch around them inside the apply costs the others 1 (FP64) to 4 % (FP32).
template <bool kSingle>
__device__ __forceinline__ void column_of(const BatchCol &c, const OffDiag &od, ConstInts ks, ConstInts ka,
                                          unsigned char *smem, double *red) {
  switch (c.L) {
    case 14: run_column<32, kSingle>(c, od, ks, ka, smem, red); break;
    case 13: run_column<16, kSingle>(c, od, ks, ka, smem, red); break;
    case 12: run_column<8, kSingle>(c, od, ks, ka, smem, red); break;
    case 11: run_column<4, kSingle>(c, od, ks, ka, smem, red); break;
    case 10: run_column<2, kSingle>(c, od, ks, ka, smem, red); break;
    default: run_column<1, kSingle>(c, od, ks, ka, smem, red); break;
  }
}

// (two waves per SIMD: 256 registers a lane)
__global__ __launch_bounds__(kBT, 2) void k_batch_chebyshev(const BatchCol *cols_g) {
  extern __shared__ unsigned char smem_raw[];  // the column, then the reductions' scratch
  // field by field through the constant address space (uniform scalar loads)
  const ConstBatchCols cc = (ConstBatchCols)cols_g + blockIdx.x;
  BatchCol c;
  c.d64 = cc->d64;
  c.d32 = cc->d32;
  c.psi0 = cc->psi0;
  c.V = cc->V;
  c.ks = cc->ks;
  c.bound_flag = cc->bound_flag;
  c.A = cc->A;
  c.ka = cc->ka;
  c.ld_psi = cc->ld_psi;
  c.ldv = cc->ldv;
  c.lda = cc->lda;
  c.f_alpha = cc->f_alpha;
  c.f_beta = cc->f_beta;
  c.f_gamma = cc->f_gamma;
  c.f_first_a = cc->f_first_a;
  c.f_first_b = cc->f_first_b;
  c.inv_e = cc->inv_e;
  c.L = cc->L;
  c.mode = cc->mode;
  c.K = cc->K;
  c.n32 = cc->n32;
  c.n_samples = cc->n_samples;
  c.b = cc->b;
  c.n_anchor = cc->n_anchor;
  const OffDiag od{(ConstDoubles)cc->xc, (ConstFlipTable)cc->flips, cc->nplain, cc->nflip};
  double *red = reinterpret_cast<double *>(smem_raw) + max(1 << c.L, kBT);
  const ConstInts ks = (ConstInts)c.ks;
  const ConstInts ka = (ConstInts)c.ka;
  if (cc->single) column_of<true>(c, od, ks, ka, smem_raw, red);
  else column_of<false>(c, od, ks, ka, smem_raw, red);
}

// ---------------------------------------------------------------------------
// Batched spectral estimates (the bound and density step of Sec. III for many realisations):
// workgroup g runs either the Lanczos recurrence of one realisation (kind 0) or the Chebyshev
// moment recurrence of one random vector of one realisation (kind 1) with the whole column on
// chip, and writes the scalars the host needs:
//   kind 0: out[j] = alpha_j, out[steps + j] = beta_j, out[2 steps] = number of steps taken,
//           out[2 steps + 1] = <start, start>;
//   kind 1: out[0] = <r, r>, out[1] = <r, T_1 r>, out[2k] = <T_k r, T_k r>,
//           out[2k + 1] = <T_(k+1) r, T_k r>  (k >= 1, indices below `steps` = M).
// ---------------------------------------------------------------------------
template <int E, bool kSingle>
__device__ __forceinline__ void run_spectral(const BatchSpec &c, const OffDiag &od, unsigned char *smem, double *red) {
  const uint32_t D = 1u << c.L;
  double *lds = reinterpret_cast<double *>(smem);
  const bool active = E > 1 || threadIdx.x < D;
  double A[E], v[E];
#pragma unroll
  for (int i = 0; i < E; ++i) {
    const uint32_t s = threadIdx.x + i * kBT;
    v[i] = active ? ld_at(c.start, s * static_cast<uint32_t>(c.ld) * 8u) : 0.0;
    A[i] = 0.0;
  }
  const double n0 = dot<E>(v, v, red);
  if (c.kind == 0) {
    // Lanczos: A = v_(j-1), v = v_j, roles swapped every step; w = H v_j - beta_(j-1) v_(j-1) - alpha_j v_j
    {
      const double inv = 1.0 / sqrt(n0);
#pragma unroll
      for (int i = 0; i < E; ++i) v[i] *= inv;
    }
    double bprev = 0.0;
    int taken = 0;
    // one step: y = v_j on entry; x = v_(j-1) becomes v_(j+1); false at the last
    auto step = [&](int j, double(&x)[E], const double(&y)[E]) -> bool {
      apply<kSingle, double, E>(y, lds, c.d64, od, D, [&](int i, double h) { set_now(x[i], h - bprev * x[i]); });
      const double alpha = dot<E>(x, y, red);
#pragma unroll
      for (int i = 0; i < E; ++i) x[i] -= alpha * y[i];
      const double beta = sqrt(fmax(dot<E>(x, x, red), 0.0));
      if (threadIdx.x == 0) {
        c.out[j] = alpha;
        c.out[c.steps + j] = beta;
      }
      taken = j + 1;
      if (!(beta > 1e-300) || j + 1 == c.steps) return false;
      const double inv = 1.0 / beta;
#pragma unroll
      for (int i = 0; i < E; ++i) x[i] *= inv;
      bprev = beta;
      return true;
    };
    for (int j = 0;; j += 2) {
      if (!step(j, A, v)) break;
      if (!step(j + 1, v, A)) break;
    }
    if (threadIdx.x == 0) {
      c.out[2 * c.steps] = static_cast<double>(taken);
      c.out[2 * c.steps + 1] = n0;
    }
    return;
  }
  // Chebyshev moments of one random vector: A = T_(k-1) r, v = T_k r, the same way
  if (threadIdx.x == 0) c.out[0] = n0;
  if (c.steps <= 1) return;
#pragma unroll
  for (int i = 0; i < E; ++i) A[i] = v[i];
  apply<kSingle, double, E>(A, lds, c.d64, od, D, [&](int i, double x) { set_now(v[i], c.inv_e * x); });
  {
    const double m1 = dot<E>(v, A, red);
    if (threadIdx.x == 0) c.out[1] = m1;
  }
  const double two_inv_e = 2.0 * c.inv_e;
  // one order: y = T_k on entry; x = T_(k-1) becomes T_(k+1); false when no moment is left
  auto order = [&](int k, double(&x)[E], const double(&y)[E]) -> bool {
    if (2 * k >= c.steps) return false;
    const double tkk = dot<E>(y, y, red);
    if (threadIdx.x == 0) c.out[2 * k] = tkk;
    if (2 * k + 1 >= c.steps) return false;
    apply<kSingle, double, E>(y, lds, c.d64, od, D, [&](int i, double h) { set_now(x[i], two_inv_e * h - x[i]); });
    const double tk1k = dot<E>(x, y, red);
    if (threadIdx.x == 0) c.out[2 * k + 1] = tk1k;
    return true;
  };
  for (int k = 1;; k += 2) {
    if (!order(k, A, v)) break;
    if (!order(k + 1, v, A)) break;
  }
}

template <bool kSingle>
__device__ __forceinline__ void spectral_of(const BatchSpec &c, const OffDiag &od, unsigned char *smem, double *red) {
  switch (c.L) {
    case 14: run_spectral<32, kSingle>(c, od, smem, red); break;
    case 13: run_spectral<16, kSingle>(c, od, smem, red); break;
    case 12: run_spectral<8, kSingle>(c, od, smem, red); break;
    case 11: run_spectral<4, kSingle>(c, od, smem, red); break;
    case 10: run_spectral<2, kSingle>(c, od, smem, red); break;
    default: run_spectral<1, kSingle>(c, od, smem, red); break;
  }
}

typedef const __attribute__((address_space(4))) BatchSpec *ConstBatchSpecs;

__global__ __launch_bounds__(kBT, 2) void k_batch_spectral(const BatchSpec *specs_g) {
  extern __shared__ unsigned char smem_raw[];  // the column, then the reductions' scratch
  const ConstBatchSpecs cs = (ConstBatchSpecs)specs_g + blockIdx.x;
  BatchSpec c;
  c.d64 = cs->d64;
  c.start = cs->start;
  c.out = cs->out;
  c.ld = cs->ld;
  c.inv_e = cs->inv_e;
  c.L = cs->L;
  c.kind = cs->kind;
  c.steps = cs->steps;
  double *red = reinterpret_cast<double *>(smem_raw) + max(1 << c.L, kBT);
  const OffDiag od{(ConstDoubles)cs->xc, (ConstFlipTable)cs->flips, cs->nplain, cs->nflip};
  if (cs->single) spectral_of<true>(c, od, smem_raw, red);
  else spectral_of<false>(c, od, smem_raw, red);
}

}  // namespace

hipError_t launch_batch_chebyshev(const BatchCol *cols, int ncols, int max_L, hipStream_t s) {
  if (ncols <= 0) return hipSuccess;
  if (max_L < 1 || max_L > 14) return hipErrorInvalidValue;
  const size_t lds = (std::max<size_t>(size_t(1) << max_L, kBT) + kBW) * sizeof(double);
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_batch_chebyshev),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_batch_chebyshev, dim3(ncols), dim3(kBT), lds, s, cols);
  return hipGetLastError();
}

hipError_t launch_batch_spectral(const BatchSpec *specs, int n, int max_L, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  if (max_L < 1 || max_L > 14) return hipErrorInvalidValue;
  const size_t lds = (std::max<size_t>(size_t(1) << max_L, kBT) + kBW) * sizeof(double);
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_batch_spectral),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_batch_spectral, dim3(n), dim3(kBT), lds, s, specs);
  return hipGetLastError();
}

}  // namespace dacp
