// C ABI and host drivers of the DACP central-eigenvalue path (gfx950).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <condition_variable>
#include <cstring>
#include <functional>
#include <tuple>
#include <map>
#include <unordered_map>
#include <new>
#include <mutex>
#include <set>
#include <numeric>
#include <type_traits>
#include <thread>
#include <utility>
#include <vector>

#include "block_cache.h"
#include "host_rules.h"
#include "internal.h"

using dacp::DevBuf;
using dacp::FlipEntry;
using dacp::StepArgs;
using dacp::to_device;
using dacp::to_host;
using dacp::BatchCol;
using dacp::BatchSpec;
using dacp::rules::AcceptResult;
using dacp::rules::Plan;
using dacp::rules::accept_rule;
using dacp::rules::anchor_orders;
using dacp::rules::central_order;
using dacp::rules::kpm_count;
using dacp::rules::make_plan;
using dacp::rules::sample_orders;
using dacp::rules::window_for_count;

namespace dacp {

bool verbose() {
  static const bool v = [] {
    const char *e = std::getenv("DACP_VERBOSE");
    return e && *e && *e != '0';
  }();
  return v;
}

void vlog(const char *fmt, ...) {
  if (!verbose()) return;
  va_list ap;
  va_start(ap, fmt);
  std::fprintf(stderr, "[dacp] ");
  std::vfprintf(stderr, fmt, ap);
  std::fprintf(stderr, "\n");
  std::fflush(stderr);
  va_end(ap);
}

AllocState &alloc_state_tl() {
  static thread_local AllocState st;
  return st;
}

namespace {
// The HIP runtime calls of the block cache (block_cache.h).
struct HipRt {
  using Stream = hipStream_t;
  using Event = hipEvent_t;
  using Err = hipError_t;
  static constexpr hipError_t ok = hipSuccess;
  static constexpr hipError_t oom = hipErrorOutOfMemory;
  hipError_t malloc(void **p, size_t n) {
    const hipError_t e = hipMalloc(p, n);
    if (e == hipErrorOutOfMemory) (void)hipGetLastError();  // clear it before the retry
    return e;
  }
  void free(void *p) { (void)hipFree(p); }
  hipError_t event_create(hipEvent_t *e) { return hipEventCreateWithFlags(e, hipEventDisableTiming); }
  hipError_t record(hipEvent_t e, hipStream_t s) { return hipEventRecord(e, s); }
  hipError_t wait(hipStream_t s, hipEvent_t e) { return hipStreamWaitEvent(s, e, 0); }
};

BlockCacheT<HipRt> &block_cache(int device) {
  static BlockCacheT<HipRt> *caches = [] {
    auto *c = static_cast<BlockCacheT<HipRt> *>(::operator new(64 * sizeof(BlockCacheT<HipRt>)));
    for (int d = 0; d < 64; ++d) new (&c[d]) BlockCacheT<HipRt>(kBlockCacheBytes);
    return c;
  }();
  return caches[device & 63];
}
}  // namespace

AllocStream::AllocStream(hipStream_t s, int device) : prev(alloc_state_tl()) {
  AllocState &st = alloc_state_tl();
  st.on = true;
  st.s = s;
  st.device = device;
}

AllocStream::~AllocStream() { alloc_state_tl() = prev; }

hipError_t pool_alloc(size_t nbytes, hipStream_t s, int device, void **p, size_t *cls) {
  HipRt rt;
  return block_cache(device).alloc(rt, nbytes, s, p, cls);
}

void pool_free(void *p, size_t cls, int device, hipStream_t s) {
  HipRt rt;
  block_cache(device).release(rt, p, cls, s);
}

dacp_status set_err(dacp_ctx ctx, dacp_status st, const std::string &msg) {
  if (ctx) ctx->err = msg;
  return st;
}

dacp_status hip_err(dacp_ctx ctx, hipError_t e, const char *what) {
  const dacp_status st = (e == hipErrorOutOfMemory) ? DACP_E_NOMEM : DACP_E_HIP;
  return set_err(ctx, st, std::string(what) + ": " + hipGetErrorString(e));
}

// Both copies are queued on the context's own stream and waited for there: a blocking copy on
// the null stream would also order against every other blocking stream of the device, which
// serialises host threads that each drive a stream of their own.
dacp_status to_host(dacp_ctx ctx, void *host, const void *dev, size_t bytes) {
  if (bytes == 0) return DACP_OK;
  DACP_HIP(ctx, hipMemcpyAsync(host, dev, bytes, hipMemcpyDeviceToHost, ctx->stream));
  DACP_HIP(ctx, hipStreamSynchronize(ctx->stream));
  return DACP_OK;
}

dacp_status to_device(dacp_ctx ctx, void *dev, const void *host, size_t bytes) {
  if (bytes == 0) return DACP_OK;
  DACP_HIP(ctx, hipMemcpyAsync(dev, host, bytes, hipMemcpyHostToDevice, ctx->stream));
  DACP_HIP(ctx, hipStreamSynchronize(ctx->stream));  // `host` may be released on return
  return DACP_OK;
}

dacp_status to_host_2d(dacp_ctx ctx, double *host, const double *dev, int64_t lddev, int64_t rows, int64_t cols) {
  if (rows <= 0 || cols <= 0) return DACP_OK;
  DevBuf tmp;
  DACP_HIP(ctx, tmp.alloc(static_cast<size_t>(rows * cols) * sizeof(double)));
  DACP_HIP(ctx, launch_copy_cols(dev, lddev, tmp.as<double>(), cols, rows, static_cast<int>(cols), ctx->stream));
  return to_host(ctx, host, tmp.p, static_cast<size_t>(rows * cols) * sizeof(double));
}

dacp_status to_device_2d(dacp_ctx ctx, double *dev, int64_t lddev, const double *host, int64_t rows, int64_t cols) {
  if (rows <= 0 || cols <= 0) return DACP_OK;
  DevBuf tmp;
  DACP_HIP(ctx, tmp.alloc(static_cast<size_t>(rows * cols) * sizeof(double)));
  DACP_TRY(to_device(ctx, tmp.p, host, static_cast<size_t>(rows * cols) * sizeof(double)));
  DACP_HIP(ctx, launch_copy_cols(tmp.as<double>(), cols, dev, lddev, rows, static_cast<int>(cols), ctx->stream));
  DACP_HIP(ctx, hipStreamSynchronize(ctx->stream));  // tmp is released on return
  return DACP_OK;
}

}  // namespace dacp

using dacp::hip_err;
using dacp::set_err;
using dacp::verbose;
using dacp::vlog;

namespace {

double now_ms() {
  return std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now().time_since_epoch()).count();
}

dacp_status ensure_red(dacp_ctx ctx, size_t partial_elems, size_t out_elems) {
  if (partial_elems > ctx->red_elems) {
    if (ctx->red) (void)hipFree(ctx->red);
    ctx->red = nullptr;
    DACP_HIP(ctx, hipMalloc(&ctx->red, partial_elems * sizeof(double)));
    ctx->red_elems = partial_elems;
  }
  if (out_elems > ctx->red_out_elems) {
    if (ctx->red_out) (void)hipFree(ctx->red_out);
    ctx->red_out = nullptr;
    DACP_HIP(ctx, hipMalloc(&ctx->red_out, out_elems * sizeof(double)));
    ctx->red_out_elems = out_elems;
  }
  return DACP_OK;
}

// Per-column dot products x_j . y_j into device memory `dev_out` (b doubles).
dacp_status coldots_dev(dacp_ctx ctx, const void *x, int64_t ldx, const void *y, int64_t ldy, int dtype, int64_t D,
                        int b, double *dev_out) {
  const int nblk = dacp::coldots_blocks(D, b);
  dacp_status st = ensure_red(ctx, static_cast<size_t>(nblk) * b, b);
  if (st) return st;
  DACP_HIP(ctx, dacp::launch_coldots(x, ldx, y, ldy, dtype, D, b, ctx->red, nblk, dev_out, ctx->stream));
  return DACP_OK;
}

// Same, result on the host (synchronises).
dacp_status coldots_host(dacp_ctx ctx, const void *x, int64_t ldx, const void *y, int64_t ldy, int dtype, int64_t D,
                         int b, double *host_out) {
  dacp_status st = ensure_red(ctx, static_cast<size_t>(dacp::coldots_blocks(D, b)) * b, b);
  if (st) return st;
  st = coldots_dev(ctx, x, ldx, y, ldy, dtype, D, b, ctx->red_out);
  if (st) return st;
  DACP_TRY(to_host(ctx, host_out, ctx->red_out, sizeof(double) * b));
  DACP_HIP(ctx, hipStreamSynchronize(ctx->stream));
  return DACP_OK;
}

// Flip table ordered for tiles of 2^log2R rows: masks inside the tile (read from LDS), masks
// entirely above it (partner row = (row0 ^ x) + r), then mixed masks; x-mask order within each.
dacp_status tile_order(dacp_ctx ctx, dacp_ham h, int log2R) {
  std::lock_guard<std::mutex> lock(h->tables_mu);
  auto &to = h->by_log2r[log2R];
  if (to.dev) return DACP_OK;
  const uint32_t lowmask = (1u << log2R) - 1u;
  std::vector<FlipEntry> lo, hi, mx;
  for (const FlipEntry &f : h->flips_host) {
    if ((f.xmask & ~lowmask) == 0) lo.push_back(f);
    else if ((f.xmask & lowmask) == 0) hi.push_back(f);
    else mx.push_back(f);
  }
  std::vector<FlipEntry> all(lo);
  all.insert(all.end(), hi.begin(), hi.end());
  all.insert(all.end(), mx.begin(), mx.end());
  DACP_HIP(ctx, hipMalloc(&to.dev, std::max<size_t>(1, all.size()) * sizeof(FlipEntry)));
  if (!all.empty())
    DACP_HIP(ctx, hipMemcpy(to.dev, all.data(), all.size() * sizeof(FlipEntry), hipMemcpyHostToDevice));
  to.nlow = static_cast<int>(lo.size());
  to.nhigh = static_cast<int>(lo.size() + hi.size());
  return DACP_OK;
}

// Flip tables for the two-pass apply split at bit lo_bits.
dacp_status split_order(dacp_ctx ctx, dacp_ham h, int lo_bits) {
  std::lock_guard<std::mutex> lock(h->tables_mu);
  auto &so = h->split[lo_bits];
  if (so.lo) return DACP_OK;
  const uint32_t lowmask = (1u << lo_bits) - 1u;
  std::vector<FlipEntry> lo, hi, mx;
  for (const FlipEntry &f : h->flips_host) {
    if ((f.xmask & ~lowmask) == 0) lo.push_back(f);
    else if ((f.xmask & lowmask) == 0) hi.push_back(f);
    else mx.push_back(f);
  }
  // sign-free (X-type, z-mask 0) flips first within each pure part: the fused kernels run them
  // in an unrolled loop without the parity sign
  auto plain_first = [](std::vector<FlipEntry> &v) {
    return static_cast<int>(std::stable_partition(v.begin(), v.end(), [](const FlipEntry &f) { return f.zmask == 0; }) -
                            v.begin());
  };
  so.nlo_plain = plain_first(lo);
  so.nhi_plain = plain_first(hi);
  hi.insert(hi.end(), mx.begin(), mx.end());
  DACP_HIP(ctx, hipMalloc(&so.lo, std::max<size_t>(1, lo.size()) * sizeof(FlipEntry)));
  DACP_HIP(ctx, hipMalloc(&so.hi, std::max<size_t>(1, hi.size()) * sizeof(FlipEntry)));
  if (!lo.empty()) DACP_HIP(ctx, hipMemcpy(so.lo, lo.data(), lo.size() * sizeof(FlipEntry), hipMemcpyHostToDevice));
  if (!hi.empty()) DACP_HIP(ctx, hipMemcpy(so.hi, hi.data(), hi.size() * sizeof(FlipEntry), hipMemcpyHostToDevice));
  so.nlo = static_cast<int>(lo.size());
  so.nhi = static_cast<int>(hi.size() - mx.size());
  so.nmix = static_cast<int>(mx.size());
  return DACP_OK;
}

// A flip that the on-chip column kernels take by bit (the others through their flip table).
bool onchip_single(const FlipEntry &f) { return f.zmask == 0 && (f.xmask & (f.xmask - 1)) == 0; }

// Tables of the on-chip column kernels (L <= 14): one coefficient per spin for the single-spin
// sign-free flips, the other flips with the sign-free ones first.
dacp_status onchip_order(dacp_ctx ctx, dacp_ham h) {
  std::lock_guard<std::mutex> lock(h->tables_mu);
  auto &oc = h->onchip;
  if (oc.xc) return DACP_OK;
  std::vector<double> xc(14, 0.0);
  std::vector<FlipEntry> rest;
  for (const FlipEntry &f : h->flips_host) {
    if (onchip_single(f)) xc[__builtin_ctz(f.xmask)] = f.coef;
    else rest.push_back(f);
  }
  const auto mid =
      std::stable_partition(rest.begin(), rest.end(), [](const FlipEntry &f) { return f.zmask == 0; });
  const int nplain = static_cast<int>(mid - rest.begin()), nflip = static_cast<int>(rest.size());
  rest.push_back(FlipEntry{0, 0, 0.0});  // the kernels load an entry ahead
  // both tables in one allocation
  const size_t bytes = 14 * sizeof(double) + rest.size() * sizeof(FlipEntry);
  double *p = nullptr;
  DACP_HIP(ctx, hipMalloc(&p, bytes));
  FlipEntry *flips = reinterpret_cast<FlipEntry *>(p + 14);
  hipError_t e = hipMemcpy(p, xc.data(), 14 * sizeof(double), hipMemcpyHostToDevice);
  if (e == hipSuccess)
    e = hipMemcpy(flips, rest.data(), rest.size() * sizeof(FlipEntry), hipMemcpyHostToDevice);
  if (e != hipSuccess) {
    (void)hipFree(p);
    return hip_err(ctx, e, "flip tables");
  }
  oc.flips = flips;
  oc.nplain = nplain;
  oc.nflip = nflip;
  oc.single = static_cast<int>(h->flips_host.size()) > nflip;
  oc.xc = p;
  return DACP_OK;
}

// Two-pass apply (low-bit tiles, then high-bit cosets), used when both tiles fit the budget.
// Returns false (nothing launched) when the shape does not allow it.
template <typename T>
bool two_pass_plan(dacp_ctx ctx, dacp_ham h, int b, int &lo_bits, int &W) {
  if (ctx->two_pass_min_L <= 0 || h->L < ctx->two_pass_min_L) return false;
  if (b & (b - 1)) return false;  // the pass kernels split elements with shifts
  const int64_t P = ctx->pass_tile_elems;
  const int L = h->L;
  lo_bits = 0;
  while (lo_bits + 1 < L && (int64_t(2) << lo_bits) * b <= P) ++lo_bits;
  const int hi_bits = L - lo_bits;
  if (lo_bits < 1 || hi_bits < 1 || (int64_t(1) << hi_bits) * b > P) return false;
  if ((int64_t(1) << lo_bits) * b < 1024) return false;  // both kernels need whole 1024-element rounds
  W = 1;
  while (W < 8 && (int64_t(2 * W) << hi_bits) * b <= P && 2 * W <= (1 << lo_bits) &&
         ((1 << lo_bits) / (2 * W)) >= 256)
    W *= 2;
  if ((int64_t(W) << hi_bits) * b < 1024) return false;
  return true;
}

// Fused alternating-split recurrence plan for a contiguous [D][g] block of FP64.  The low
// tile (2^lo_bits rows) and the high tile (W adjacent rows x 2^(L - lo_bits) cosets) each hold
// 2, 4 or 8 16-byte vectors per thread and at most rec_tile elements (64 KB of LDS), the high
// tile's contiguous runs of W rows fill whole 128-byte lines where possible, and no flip mask
// straddles bit lo_bits.
bool fused_plan(dacp_ctx ctx, dacp_ham h, int g, int &lo_bits, int &W, int esize) {
  if (!ctx->fused_rec || ctx->two_pass_min_L <= 0 || h->L < ctx->two_pass_min_L) return false;
  if ((g & (g - 1)) || g < 2 || g * esize < 16) return false;
  // the kernels address a block with 32-bit byte offsets
  if (h->D * g * static_cast<int64_t>(esize) >= (int64_t(1) << 32)) return false;
  const int L = h->L;
  // tile bytes: at most rec_tile FP64 elements (64 KB of LDS)
  const int64_t Pb = std::min<int64_t>(ctx->rec_tile_elems, 8192) * 8;
  const int64_t nt = ctx->rec_threads;
  auto ok_tile = [&](int64_t nel) {
    const int64_t bytes = nel * esize;
    const int64_t per = bytes / 16 / nt;  // 16-byte vectors per thread
    return bytes <= Pb && bytes % (16 * nt) == 0 && (per == 1 || per == 2 || per == 4) && bytes >= 8192;
  };
  int w0 = ctx->rec_hi_w;
  if (w0 <= 0) {
    w0 = 1;
    while (w0 * g * esize < 128 && w0 < 8) w0 *= 2;
  }
  const uint32_t all = (L >= 32) ? 0xffffffffu : ((1u << L) - 1u);
  for (W = w0; W >= 1; W /= 2) {
    for (lo_bits = L - 1; lo_bits >= 1; --lo_bits) {
      const int hi_bits = L - lo_bits;
      if ((int64_t(1) << lo_bits) < W) break;
      const int64_t nlo = (int64_t(1) << lo_bits) * g, nhi = (int64_t(W) << hi_bits) * g;
      if (!ok_tile(nlo) || !ok_tile(nhi)) continue;
      const uint32_t lowmask = (1u << lo_bits) - 1u;
      bool straddle = false;
      for (const FlipEntry &f : h->flips_host)
        if ((f.xmask & lowmask) && (f.xmask & ~lowmask & all)) straddle = true;
      if (straddle) continue;
      return true;
    }
  }
  return false;
}

// Column groups of a recurrence over b columns, `g` columns wanted per group (rules::column_plan): what the
// launch that starts at column c0 advances.  A shape without a fused plan keeps its width and runs one
// group at a time.
struct ColGroups : dacp::rules::ColumnPlan {
  int b;
  int cols(int c0) const { return c0 < b - tail ? std::min(g * per, b - tail - c0) : tail; }
  int width(int c0) const { return c0 >= b - tail ? tail_w : fused ? g : cols(c0); }
  int groups(int c0) const { return c0 < b - tail && fused ? (cols(c0) + g - 1) / g : 1; }
  size_t elems(int64_t D) const { return static_cast<size_t>(D) * g * per; }
};
// `blocks` live [D][g] blocks of up to the largest of `esizes` bytes an element; filter: its launches do
// two applies.
ColGroups column_groups(dacp_ctx ctx, dacp_ham h, int b, int g, int blocks, std::initializer_list<int> esizes,
                        bool filter = false) {
  auto fused = [&](int w) {
    for (int e : esizes) {
      int lo_bits = 0, hw = 1;
      if (!fused_plan(ctx, h, w, lo_bits, hw, e)) return false;
    }
    return true;
  };
  ColGroups cg;
  static_cast<dacp::rules::ColumnPlan &>(cg) = dacp::rules::column_plan(
      h->D, b, g, static_cast<int64_t>(blocks) * *std::max_element(esizes.begin(), esizes.end()), esizes.size() > 1, filter, fused);
  cg.b = b;
  return cg;
}

// y = alpha H x + beta u + gamma z (+ FP64 copy into st), columns split in chunks of <= 2048.
template <typename T>
dacp_status step(dacp_ctx ctx, dacp_ham h, int b, const T *x, int64_t ldx, T *y, int64_t ldy, T alpha,
                 const T *u = nullptr, int64_t ldu = 0, T beta = T(0), const T *z = nullptr, int64_t ldz = 0,
                 T gamma = T(0), double *st = nullptr, int64_t ldst = 0, int role = 0) {
  const int64_t D = h->D;
  int lo_bits = 0, W = 1;
  if (x != y && two_pass_plan<T>(ctx, h, b, lo_bits, W)) {
    dacp_status sst = split_order(ctx, h, lo_bits);
    if (sst) return sst;
    const auto &so = h->split[lo_bits];
    StepArgs<T> a;
    a.x = x;
    a.ldx = ldx;
    a.y = y;
    a.ldy = ldy;
    a.u = u;
    a.ldu = ldu;
    a.z = z;
    a.ldz = ldz;
    a.st = nullptr;
    a.ldst = 0;
    a.alpha = alpha;
    a.beta = beta;
    a.gamma = gamma;
    a.diag = std::is_same<T, double>::value ? reinterpret_cast<const T *>(h->d64) : reinterpret_cast<const T *>(h->d32);
    a.flips = so.lo;
    a.nflip = so.nlo;
    a.nlow = so.nlo;
    a.nhigh = so.nlo;
    a.b = b;
    a.log2R = lo_bits;
    a.ntiles = static_cast<int>(D >> lo_bits);
    a.xcd_remap = 0;
    DACP_HIP(ctx, dacp::launch_step_lo<T>(a, ctx->stream, role));
    dacp::HiArgs<T> hb;
    hb.x = x;
    hb.ldx = ldx;
    hb.y = y;
    hb.ldy = ldy;
    hb.st = st;
    hb.ldst = ldst;
    hb.alpha = alpha;
    hb.flips = so.hi;
    hb.nhi = so.nhi;
    hb.nflip = so.nhi + so.nmix;
    hb.b = b;
    hb.lo_bits = lo_bits;
    hb.hi_bits = h->L - lo_bits;
    hb.W = W;
    hb.ntiles = (1 << lo_bits) / W;
    DACP_HIP(ctx, dacp::launch_step_hi<T>(hb, ctx->stream, role));
    return DACP_OK;
  }
  for (int c0 = 0; c0 < b; c0 += 2048) {
    const int bc = std::min(2048, b - c0);
    int log2R = 0;
    // rows per tile: R * bc <= tile, R <= D, and R * ldx * sizeof(T) < 2^31 (32-bit in-tile offsets)
    while ((int64_t(2) << log2R) <= D && (int64_t(2) << log2R) * bc <= ctx->tile_elems &&
           (int64_t(2) << log2R) * ldx * static_cast<int64_t>(sizeof(T)) < (int64_t(1) << 31))
      ++log2R;
    StepArgs<T> a;
    a.x = x + c0;
    a.ldx = ldx;
    a.y = y + c0;
    a.ldy = ldy;
    a.u = u ? u + c0 : nullptr;
    a.ldu = ldu;
    a.z = z ? z + c0 : nullptr;
    a.ldz = ldz;
    a.st = st ? st + c0 : nullptr;
    a.ldst = ldst;
    a.alpha = alpha;
    a.beta = beta;
    a.gamma = gamma;
    a.diag = std::is_same<T, double>::value ? reinterpret_cast<const T *>(h->d64) : reinterpret_cast<const T *>(h->d32);
    dacp_status ost = tile_order(ctx, h, log2R);
    if (ost) return ost;
    a.flips = h->by_log2r[log2R].dev;
    a.nflip = static_cast<int>(h->flips_host.size());
    a.nlow = h->by_log2r[log2R].nlow;
    a.nhigh = h->by_log2r[log2R].nhigh;
    a.b = bc;
    a.log2R = log2R;
    a.ntiles = static_cast<int>(D >> log2R);
    a.xcd_remap = (a.ntiles % 8 == 0 && a.ntiles >= 64) ? 1 : 0;
    DACP_HIP(ctx, dacp::launch_step<T>(a, ctx->stream, role));
  }
  return DACP_OK;
}

struct Timer {
  dacp_ctx ctx;
  hipEvent_t a, b;
  explicit Timer(dacp_ctx c) : ctx(c) {
    (void)hipEventCreate(&a);
    (void)hipEventCreate(&b);
  }
  ~Timer() {
    (void)hipEventDestroy(a);
    (void)hipEventDestroy(b);
  }
  void start() { (void)hipEventRecord(a, ctx->stream); }
  double stop_ms() {
    (void)hipEventRecord(b, ctx->stream);
    (void)hipEventSynchronize(b);
    float ms = 0.f;
    (void)hipEventElapsedTime(&ms, a, b);
    return ms;
  }
};

// ------------------------------------------------------- on-chip columns
// Up to kOnChipL spins a column fits one compute unit, and a recurrence runs there whole, a
// workgroup per column (batch.hip): one launch, where a step through memory is one to four
// launches of about 5 us each whatever the size.  Taken where it is the faster route (rules::onchip_pays:
// flips of two spins or with a sign cost a sweep of the column each) and the column's 32-bit byte
// offsets reach, over `applies` applies to each of b columns of a block with row stride ld.
constexpr int kOnChipL = 14;
bool onchip_fits(dacp_ctx ctx, dacp_ham h, int b, int64_t ld, double applies, double extra_us = 0.0) {
  if (h->L > kOnChipL || h->D * std::max<int64_t>(b, ld) * 8 >= (int64_t(1) << 32)) return false;
  return dacp::rules::onchip_pays(h->L, h->flip_counts, b, ctx->num_cus, applies, extra_us);
}

// A column's table entry without its buffers: h's tables and the recurrences' coefficients (a > 0:
// the filter's too).
BatchCol onchip_col(dacp_ham h, int mode, double e_b, double a) {
  BatchCol c;
  std::memset(&c, 0, sizeof(c));
  c.xc = h->onchip.xc;
  c.flips = h->onchip.flips;
  c.nflip = h->onchip.nflip;
  c.nplain = h->onchip.nplain;
  c.single = h->onchip.single;
  c.d64 = h->d64;
  c.d32 = h->d32;
  c.L = h->L;
  c.mode = mode;
  c.inv_e = 1.0 / e_b;
  if (a > 0.0) {
    const double e_c = 0.5 * (e_b * e_b + a * a), e_0 = 0.5 * (e_b * e_b - a * a);
    const double rho = std::exp(std::acosh(1.0 + 2.0 * a * a / (e_b * e_b - a * a)));
    c.f_alpha = 2.0 / (e_0 * rho);
    c.f_beta = -2.0 * e_c / (e_0 * rho);
    c.f_gamma = -1.0 / (rho * rho);
    c.f_first_a = 1.0 / (e_0 * rho);
    c.f_first_b = -e_c / (e_0 * rho);
  }
  return c;
}

// The evolution of all b columns from psi_e (D x b) on chip: panels at 0 and the sample orders ks into
// V and, with anchors, the panels of the anchor orders into abuf (row stride lda).  Returns the norm
// check's outcome as run_basis does (`what` names the entry point).
dacp_status onchip_evolve(dacp_ctx ctx, dacp_ham h, double e_bound, int b, const double *psi_e,
                          const std::vector<int64_t> &ks, double *V, int64_t ldv, const std::vector<int64_t> *anchors,
                          double *abuf, int64_t lda, const char *what) {
  DACP_TRY(onchip_order(ctx, h));
  std::vector<int> tab(ks.begin(), ks.end());
  const int na = anchors ? static_cast<int>(anchors->size()) : 0;
  if (anchors) tab.insert(tab.end(), anchors->begin(), anchors->end());
  tab.push_back(dacp::kBatchNoFlag);
  DevBuf dtab, dcols;
  DACP_HIP(ctx, dtab.alloc(tab.size() * sizeof(int)));
  DACP_HIP(ctx, dcols.alloc(sizeof(BatchCol) * b));
  std::vector<BatchCol> cols;
  for (int j = 0; j < b; ++j) {
    BatchCol c = onchip_col(h, dacp::kBatchEvolve, e_bound, 0.0);
    c.psi0 = psi_e + j;
    c.ld_psi = b;
    c.V = V + j;
    c.ldv = ldv;
    c.b = b;
    c.ks = dtab.as<int>();
    c.n_samples = static_cast<int>(ks.size());
    c.n_anchor = na;
    c.ka = dtab.as<int>() + ks.size();
    c.A = abuf ? abuf + j : nullptr;
    c.lda = lda;
    c.bound_flag = dtab.as<int>() + ks.size() + na;
    cols.push_back(c);
  }
  DACP_TRY(to_device(ctx, dtab.p, tab.data(), tab.size() * sizeof(int)));
  DACP_TRY(to_device(ctx, dcols.p, cols.data(), sizeof(BatchCol) * b));
  DACP_HIP(ctx, dacp::launch_batch_chebyshev(dcols.as<BatchCol>(), b, h->L, ctx->stream));
  int flag = 0;
  DACP_TRY(to_host(ctx, &flag, cols[0].bound_flag, sizeof(int)));
  if (flag == dacp::kBatchNoFlag) return DACP_OK;
  if (flag & 1) return set_err(ctx, DACP_E_NUMERIC, std::string(what) + ": non-finite evolved state");
  return set_err(ctx, DACP_E_BOUNDS, std::string(what) + ": |T_k(H/e_bound)| grew above 1; e_bound is below ||H||");
}

// ------------------------------------------------------------- filter core
// Damped recurrence: with rho = exp(theta_0), theta_0 = arccosh(1 + 2a^2/(E_b^2 - a^2))
// the growth rate of the band-centre component, the kernels carry
// T^_k = T_k / rho^k, which obeys T^_{k+1} = (2/rho) F T^_k - (1/rho^2) T^_{k-1};
// the normalised output is unchanged and FP32 never overflows.
struct FilterCoefs {
  double e_c, e_0, rho;
};

template <typename T>
dacp_status filter_first(dacp_ctx ctx, dacp_ham h, int b, const FilterCoefs &fc, const T *psi, T *t1, T *w) {
  dacp_status st = step<T>(ctx, h, b, psi, b, w, b, T(1), nullptr, 0, T(0), nullptr, 0, T(0), nullptr, 0, 1);
  if (st) return st;
  return step<T>(ctx, h, b, w, b, t1, b, T(1.0 / (fc.e_0 * fc.rho)), psi, b, T(-fc.e_c / (fc.e_0 * fc.rho)), nullptr, 0,
                 T(0), nullptr, 0, 1);
}

// Advance (A = T^_{k-1}, B = T^_k) by `nsteps`; on return B holds the newest.
template <typename T>
dacp_status filter_steps(dacp_ctx ctx, dacp_ham h, int b, const FilterCoefs &fc, T *&A, T *&B, T *w, int nsteps) {
  const T alpha = T(2.0 / (fc.e_0 * fc.rho));
  const T beta = T(-2.0 * fc.e_c / (fc.e_0 * fc.rho));
  const T gamma = T(-1.0 / (fc.rho * fc.rho));
  for (int k = 0; k < nsteps; ++k) {
    dacp_status st = step<T>(ctx, h, b, B, b, w, b, T(1), nullptr, 0, T(0), nullptr, 0, T(0), nullptr, 0, 1);
    if (st) return st;
    st = step<T>(ctx, h, b, w, b, A, b, alpha, B, b, beta, A, b, gamma, nullptr, 0, 1);
    if (st) return st;
    std::swap(A, B);
  }
  return DACP_OK;
}

// The filter orders as one chain of fused split kernels (see RecArgs).  Per order, the low tile
// kernel completes w = H T^_k and starts the partial of T^_{k+1} = alpha H w + beta T^_k +
// gamma T^_{k-1}; the high coset kernel completes T^_{k+1} and starts the partial of the next w.
// Same recurrence as filter_steps, with 9 block streams per order instead of two full applies
// with global gathers.  A, B, W and Pp hold `groups` [D][b] blocks each.  `done` stays false, and nothing is
// launched, when the shape has no fused plan.
template <typename T>
dacp_status filter_steps_fused(dacp_ctx ctx, dacp_ham h, int b, int groups, const FilterCoefs &fc, T *&A, T *&B, T *W,
                               T *Pp, int nsteps, bool &done) {
  done = false;
  int lo_bits = 0, hw = 1;
  if (nsteps < 1 || !fused_plan(ctx, h, b, lo_bits, hw, static_cast<int>(sizeof(T)))) return DACP_OK;
  dacp_status st = split_order(ctx, h, lo_bits);
  if (st) return st;
  const auto &so = h->split[lo_bits];
  const int64_t D = h->D;
  hipStream_t s = ctx->stream;
  // partial of w_1 = H B: the high half, Pp = Hi B
  DACP_HIP(ctx, hipMemsetAsync(Pp, 0, static_cast<size_t>(D) * b * groups * sizeof(T), s));
  for (int y = 0; y < groups; ++y) {
    dacp::HiArgs<T> hb;
    std::memset(&hb, 0, sizeof(hb));
    hb.x = B + y * D * b;
    hb.ldx = b;
    hb.y = Pp + y * D * b;
    hb.ldy = b;
    hb.alpha = T(1);
    hb.flips = so.hi;
    hb.nhi = so.nhi;
    hb.nflip = so.nhi;
    hb.b = b;
    hb.lo_bits = lo_bits;
    hb.hi_bits = h->L - lo_bits;
    hb.W = hw;
    hb.ntiles = (1 << lo_bits) / hw;
    DACP_HIP(ctx, dacp::launch_step_hi<T>(hb, s, 1));
  }
  const T alpha = T(2.0 / (fc.e_0 * fc.rho));
  const T beta = T(-2.0 * fc.e_c / (fc.e_0 * fc.rho));
  const T gamma = T(-1.0 / (fc.rho * fc.rho));
  dacp::RecArgs<T> ra;
  std::memset(&ra, 0, sizeof(ra));
  ra.groups = groups;
  ra.gstride = D * b;
  ra.diag = std::is_same<T, double>::value ? reinterpret_cast<const T *>(h->d64) : reinterpret_cast<const T *>(h->d32);
  ra.b = b;
  ra.lo_bits = lo_bits;
  ra.hi_bits = h->L - lo_bits;
  ra.W = hw;
  ra.threads = ctx->rec_threads;
  ra.grid = ctx->rec_persist * ctx->num_cus;
  ra.p = Pp;
  for (int k = 0; k < nsteps; ++k) {
    // low: W = Pp + (D + Lo) B;  Pp <- alpha (D + Lo) W + beta B + gamma A
    ra.tcur = B;
    ra.tnew = W;
    ra.old = A;
    ra.a_fin = T(1);
    ra.a_start = alpha;
    ra.b_cur = beta;
    ra.c_old = gamma;
    ra.flips = so.lo;
    ra.nflip = so.nlo;
    ra.nplain = so.nlo_plain;
    ra.ntiles = static_cast<int>(D >> lo_bits);
    ra.xcd_remap = ((ctx->rec_xcd & 1) && ra.ntiles % 8 == 0) ? 1 : 0;
    DACP_HIP(ctx, dacp::launch_rec_lo<T>(ra, s));
    // high: A = Pp + alpha Hi W (the new order, over T^_{k-1});  Pp <- Hi A
    ra.tcur = W;
    ra.tnew = A;
    ra.old = nullptr;
    ra.a_fin = alpha;
    ra.a_start = T(1);
    ra.b_cur = T(0);
    ra.c_old = T(0);
    ra.flips = so.hi;
    ra.nflip = so.nhi;
    ra.nplain = so.nhi_plain;
    ra.ntiles = (1 << lo_bits) / hw;
    ra.xcd_remap = ((ctx->rec_xcd & 2) && ra.ntiles % 8 == 0) ? 1 : 0;
    DACP_HIP(ctx, dacp::launch_rec_hi<T>(ra, s));
    std::swap(A, B);
  }
  done = true;
  return DACP_OK;
}

dacp_status normalise_cols(dacp_ctx ctx, double *x, int64_t D, int b) {
  dacp_status st = ensure_red(ctx, static_cast<size_t>(dacp::coldots_blocks(D, b)) * b, b);
  if (st) return st;
  std::vector<double> nrm(b);
  st = coldots_host(ctx, x, b, x, b, DACP_F64, D, b, nrm.data());
  if (st) return st;
  for (int j = 0; j < b; ++j)
    if (!(nrm[j] > 0.0) || !std::isfinite(nrm[j]))
      return set_err(ctx, DACP_E_NUMERIC, "filtered column has zero or non-finite norm");
  DACP_HIP(ctx, dacp::launch_colscale(x, b, D, b, ctx->red_out, ctx->stream));
  return DACP_OK;
}

// Filter `groups` contiguous [D][g] groups of start columns (FP32 part, then FP64 steps); the
// newest recurrence term ends in `out` (same layout, FP64, not normalised).  More than one group
// only for a shape with fused plans.
dacp_status filter_group(dacp_ctx ctx, dacp_ham h, int g, int groups, const FilterCoefs &fc, int K, int tail_in,
                         int precision, const double *psi, double *out) {
  const int64_t D = h->D, DG = D * groups;
  const size_t blk = static_cast<size_t>(DG) * g;
  if (K == 0) {
    DACP_HIP(ctx, dacp::launch_copy_cols(psi, g, out, g, DG, g, ctx->stream));
    return DACP_OK;
  }
  DevBuf a64, w64, b64;
  DACP_HIP(ctx, a64.alloc(blk * sizeof(double)));
  DACP_HIP(ctx, w64.alloc(blk * sizeof(double)));
  DACP_HIP(ctx, b64.alloc(blk * sizeof(double)));
  double *A = a64.as<double>(), *B = b64.as<double>();
  int tail = (precision == DACP_F32) ? std::max(0, std::min(tail_in, K)) : K;
  const int n32 = K - tail;  // orders reached in FP32
  dacp_status st = DACP_OK;
  if (n32 >= 1) {
    DevBuf a32, b32, w32, p32;
    DACP_HIP(ctx, a32.alloc(blk * sizeof(float)));
    DACP_HIP(ctx, b32.alloc(blk * sizeof(float)));
    DACP_HIP(ctx, w32.alloc(blk * sizeof(float)));
    DACP_HIP(ctx, p32.alloc(blk * sizeof(float)));
    DACP_HIP(ctx, dacp::launch_convert_f64_to_f32(psi, g, p32.as<float>(), g, DG, g, ctx->stream));
    float *A32 = a32.as<float>(), *B32 = b32.as<float>();
    DACP_HIP(ctx, dacp::launch_convert_f64_to_f32(psi, g, A32, g, DG, g, ctx->stream));
    for (int y = 0; y < groups; ++y) {
      st = filter_first<float>(ctx, h, g, fc, p32.as<float>() + y * D * g, B32 + y * D * g, w32.as<float>() + y * D * g);
      if (st) return st;
    }
    bool fused = false;
    if (n32 - 1 >= 1) {
      DevBuf q32;
      DACP_HIP(ctx, q32.alloc(blk * sizeof(float)));
      st = filter_steps_fused<float>(ctx, h, g, groups, fc, A32, B32, w32.as<float>(), q32.as<float>(), n32 - 1, fused);
      if (st) return st;
      if (fused) DACP_HIP(ctx, hipStreamSynchronize(ctx->stream));  // q32 is released at scope end
    }
    if (!fused && n32 - 1 >= 1) {  // one group
      st = filter_steps<float>(ctx, h, g, fc, A32, B32, w32.as<float>(), n32 - 1);
      if (st) return st;
    }
    DACP_HIP(ctx, dacp::launch_convert_f32_to_f64(A32, g, A, g, DG, g, ctx->stream));
    DACP_HIP(ctx, dacp::launch_convert_f32_to_f64(B32, g, B, g, DG, g, ctx->stream));
    DACP_HIP(ctx, hipStreamSynchronize(ctx->stream));  // FP32 buffers are released at scope end
  } else {
    DACP_HIP(ctx, dacp::launch_copy_cols(psi, g, A, g, DG, g, ctx->stream));
    for (int y = 0; y < groups; ++y) {
      st = filter_first<double>(ctx, h, g, fc, psi + y * D * g, B + y * D * g, w64.as<double>() + y * D * g);
      if (st) return st;
    }
    tail = K - 1;
  }
  bool fused = false;
  DevBuf q64;
  if (tail >= 1) {
    DACP_HIP(ctx, q64.alloc(blk * sizeof(double)));
    st = filter_steps_fused<double>(ctx, h, g, groups, fc, A, B, w64.as<double>(), q64.as<double>(), tail, fused);
    if (st) return st;
  }
  if (!fused && tail >= 1) {  // one group
    st = filter_steps<double>(ctx, h, g, fc, A, B, w64.as<double>(), tail);
    if (st) return st;
  }
  DACP_HIP(ctx, dacp::launch_copy_cols(B, g, out, g, DG, g, ctx->stream));
  DACP_HIP(ctx, hipStreamSynchronize(ctx->stream));
  return DACP_OK;
}

// Column-group width for the recurrences: the columns are independent, and a narrow group keeps
// the recurrence's working set (two or three [D][g] blocks) inside the 256 MB Infinity Cache.
int recurrence_group(dacp_ctx ctx, dacp_ham h, int b) {
  if (h->L >= 15 && b > ctx->group_default) return ctx->group_default;
  return b;
}

dacp_status run_filter(dacp_ctx ctx, dacp_ham h, const dacp_filter_params *p, const double *start, double *psi_out) {
  const int64_t D = h->D;
  const int b = p->b;
  if (b < 1 || p->K < 0 || !(p->a > 0.0) || !(p->e_bound > p->a) || !psi_out)
    return set_err(ctx, DACP_E_INVALID, "filter: need b >= 1, K >= 0, 0 < a < e_bound, psi_out");
  if (p->precision != DACP_F64 && p->precision != DACP_F32)
    return set_err(ctx, DACP_E_INVALID, "filter: precision must be DACP_F64 or DACP_F32");
  FilterCoefs fc;
  fc.e_c = 0.5 * (p->e_bound * p->e_bound + p->a * p->a);
  fc.e_0 = 0.5 * (p->e_bound * p->e_bound - p->a * p->a);
  fc.rho = std::exp(std::acosh(1.0 + 2.0 * p->a * p->a / (p->e_bound * p->e_bound - p->a * p->a)));
  DevBuf s0;
  const double *psi = start;
  if (!psi) {
    DACP_HIP(ctx, s0.alloc(static_cast<size_t>(D) * b * sizeof(double)));
    DACP_HIP(ctx, dacp::launch_philox_gauss(s0.as<double>(), D, b, p->seed, ctx->stream));
    psi = s0.as<double>();
  }
  if (p->K > 0 && onchip_fits(ctx, h, b, b, 2.0 * p->K)) {
    DACP_TRY(onchip_order(ctx, h));
    const int tail = p->precision == DACP_F32 ? std::max(0, std::min(p->fp64_tail, p->K)) : p->K;
    std::vector<BatchCol> cols;
    for (int j = 0; j < b; ++j) {
      BatchCol c = onchip_col(h, dacp::kBatchFilter, p->e_bound, p->a);
      c.psi0 = psi + j;
      c.ld_psi = b;
      c.V = psi_out + j;
      c.ldv = b;
      c.b = b;
      c.K = p->K;
      c.n32 = p->K - tail;
      cols.push_back(c);
    }
    DevBuf dcols;
    DACP_HIP(ctx, dcols.alloc(sizeof(BatchCol) * b));
    DACP_TRY(to_device(ctx, dcols.p, cols.data(), sizeof(BatchCol) * b));
    DACP_HIP(ctx, dacp::launch_batch_chebyshev(dcols.as<BatchCol>(), b, h->L, ctx->stream));
    DACP_TRY(normalise_cols(ctx, psi_out, D, b));
    DACP_HIP(ctx, hipStreamSynchronize(ctx->stream));
    return DACP_OK;
  }
  const int gf = p->precision == DACP_F32 ? ctx->filter_group_f32 : ctx->filter_group_f64;
  // four live blocks: T_(k-1), T_k, w and the partial
  const int gt = (h->L >= 15 && b > gf) ? gf : b;
  const ColGroups cg = p->precision == DACP_F32 ? column_groups(ctx, h, b, gt, 4, {4, 8}, true)
                                                : column_groups(ctx, h, b, gt, 4, {8}, true);
  DevBuf gin, gout;
  DACP_HIP(ctx, gin.alloc(cg.elems(D) * sizeof(double)));
  DACP_HIP(ctx, gout.alloc(cg.elems(D) * sizeof(double)));
  for (int g0 = 0; g0 < b; g0 += cg.cols(g0)) {
    const int nc = cg.cols(g0), gw = cg.width(g0), groups = cg.groups(g0);
    DACP_HIP(ctx, dacp::launch_split_cols(psi + g0, b, nc, gin.as<double>(), D, gw, groups, ctx->stream));
    dacp_status st = filter_group(ctx, h, gw, groups, fc, p->K, p->fp64_tail, p->precision, gin.as<double>(),
                                  gout.as<double>());
    if (st) return st;
    DACP_HIP(ctx, dacp::launch_join_cols(gout.as<double>(), D, gw, groups, psi_out + g0, b, nc, ctx->stream));
    vlog("filter columns %d..%d of %d done", g0, g0 + nc, b);
  }
  dacp_status st = normalise_cols(ctx, psi_out, D, b);
  if (st) return st;
  DACP_HIP(ctx, hipStreamSynchronize(ctx->stream));
  return DACP_OK;
}

// ------------------------------------------------------------- basis core
struct EvolStats {
  int64_t steps = 0, launches = 0;
  double kernel_ms = 0.0;
  int group = 0;
};

// A captured run of launches, replayed with one hipGraphLaunch.  capture(n, launch) records
// launch(j, stream) for j = 0 .. n-1 on a private stream; any failure leaves no graph (failed set)
// and the caller launches one by one.  Only kernel launches are recorded.
struct GraphRun {
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
  bool failed = false;
  template <typename F>
  void capture(int n, F launch) {
    hipStream_t cs = nullptr;
    if (hipStreamCreateWithFlags(&cs, hipStreamNonBlocking) != hipSuccess) {
      failed = true;
      return;
    }
    bool ok = hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal) == hipSuccess;
    for (int j = 0; ok && j < n; ++j) ok = launch(j, cs) == hipSuccess;
    hipGraph_t g = nullptr;
    const bool ended = hipStreamEndCapture(cs, &g) == hipSuccess;
    if (ok && ended && g && hipGraphInstantiate(&exec, g, nullptr, nullptr, 0) == hipSuccess) {
      graph = g;
    } else {
      if (g) (void)hipGraphDestroy(g);
      exec = nullptr;
      failed = true;
      (void)hipGetLastError();
    }
    (void)hipStreamDestroy(cs);
  }
  ~GraphRun() {
    if (exec) (void)hipGraphExecDestroy(exec);
    if (graph) (void)hipGraphDestroy(graph);
  }
};

// Chebyshev evolution T_{k+1}(G) = 2 G T_k - T_{k-1} (Sec. II.B) of ncols columns from T_0 (in A) up
// to T_kmax, G = H inv_e.  A, B and P hold `groups` [D][gw] blocks, block after block (more than one,
// or columns past ncols, only for a shape with a fused plan).
//   store_of(k)       device pointer (row stride ldst) that the kernel writing T_k also fills with an
//                     FP64 copy of its ncols columns, or null
//   visit(k, T_k, T_{k-1})  called once T_k is complete (the blocks of A's layout; T_{k-1} null at
//                     k = 0) for every k with want(k); it may queue work on the context stream that
//                     reads them (queued before their buffers are reused)
//   events(k1, k2)    whether a store or a visit falls on k1..k2 (such steps are not replayed from a
//                     captured graph)
dacp_status evolve_group(dacp_ctx ctx, dacp_ham h, double inv_e, int64_t kmax, int gw, int groups, int ncols,
                         double *A, double *B, double *Pp, const std::function<double *(int64_t)> &store_of, int64_t ldst,
                         const std::function<bool(int64_t)> &want,
                         const std::function<dacp_status(int64_t, const double *, const double *)> &visit,
                         const std::function<bool(int64_t, int64_t)> &events, int64_t &launches) {
  const int64_t D = h->D;
  double *const A0 = A;
  if (want(0)) DACP_TRY(visit(0, A, nullptr));
  if (kmax < 1) return DACP_OK;
  dacp_status st = DACP_OK;
  const int64_t blk = D * gw;
  for (int y = 0; y < groups; ++y) {
    double *const s1 = store_of(1);
    const int nc = std::min(gw, ncols - y * gw);  // a block with zero columns stores by a copy
    double *const sy = (s1 && nc == gw) ? s1 + y * gw : nullptr;
    st = step<double>(ctx, h, gw, A + y * blk, gw, B + y * blk, gw, inv_e, nullptr, 0, 0.0, nullptr, 0, 0.0, sy, ldst, 2);
    if (st) return st;
    if (s1 && !sy) DACP_HIP(ctx, dacp::launch_copy_cols(B + y * blk, gw, s1 + y * gw, ldst, D, nc, ctx->stream));
    ++launches;
  }
  if (want(1)) DACP_TRY(visit(1, B, A));
  const int64_t report_every = std::max<int64_t>(1, kmax / 8);
  int lo_bits = 0, hw = 1;
  if (kmax > 1 && Pp && fused_plan(ctx, h, gw, lo_bits, hw, 8)) {
    // P_2 = (2/E)(D + Lo) T_1 - T_0 by the low-bit pass, then alternate high / low fused kernels.
    st = split_order(ctx, h, lo_bits);
    if (st) return st;
    const auto &so = h->split[lo_bits];
    for (int y = 0; y < groups; ++y) {
      StepArgs<double> sa;
      std::memset(&sa, 0, sizeof(sa));
      sa.x = B + y * blk;
      sa.ldx = gw;
      sa.y = Pp + y * blk;
      sa.ldy = gw;
      sa.z = A + y * blk;
      sa.ldz = gw;
      sa.alpha = 2.0 * inv_e;
      sa.gamma = -1.0;
      sa.diag = h->d64;
      sa.flips = so.lo;
      sa.nflip = so.nlo;
      sa.nlow = so.nlo;
      sa.nhigh = so.nlo;
      sa.b = gw;
      sa.log2R = lo_bits;
      sa.ntiles = static_cast<int>(D >> lo_bits);
      DACP_HIP(ctx, dacp::launch_step_lo<double>(sa, ctx->stream, 2));
    }
    dacp::RecArgs<double> ra;
    std::memset(&ra, 0, sizeof(ra));
    ra.groups = groups;
    ra.gstride = blk;
    ra.ldst = ldst;
    ra.st_cols = ncols;
    ra.a_fin = ra.a_start = 2.0 * inv_e;
    ra.b_cur = -1.0;
    ra.diag = h->d64;
    ra.b = gw;
    ra.lo_bits = lo_bits;
    ra.hi_bits = h->L - lo_bits;
    ra.W = hw;
    ra.threads = ctx->rec_threads;
    ra.grid = ctx->rec_persist * ctx->num_cus;
    ra.p = Pp;
    // one step: T_{k+1} from T_k (tcur) and the partial; T_{k+1} overwrites T_{k-1} (tnew)
    auto launch_step = [&](int64_t k, double *tcur, double *tnew, double *stv, hipStream_t s) -> hipError_t {
      ra.tcur = tcur;
      ra.tnew = tnew;
      ra.st = stv;
      if ((k % 2) == 1) {
        ra.flips = so.hi;
        ra.nflip = so.nhi;
        ra.nplain = so.nhi_plain;
        ra.ntiles = (1 << lo_bits) / hw;
        ra.xcd_remap = ((ctx->rec_xcd & 2) && ra.ntiles % 8 == 0) ? 1 : 0;
        return dacp::launch_rec_hi<double>(ra, s);
      }
      ra.flips = so.lo;
      ra.nflip = so.nlo;
      ra.nplain = so.nlo_plain;
      ra.ntiles = static_cast<int>(D >> lo_bits);
      ra.xcd_remap = ((ctx->rec_xcd & 1) && ra.ntiles % 8 == 0) ? 1 : 0;
      return dacp::launch_rec_lo<double>(ra, s);
    };
    // Below 2^19 rows a launch is a few microseconds and its issue cost shows, so runs of
    // rec_graph steps without a store or a visit (a high/low period starting on a high step, the
    // buffers then in their starting roles) replay one captured graph.
    GraphRun graph;
    const int gsteps = (D < (int64_t(1) << 19) && kmax > 4 * ctx->rec_graph) ? ctx->rec_graph : 0;
    double *const B0 = B;
    for (int64_t k = 1; k < kmax;) {
      if (gsteps > 0 && (k % 2) == 1 && k + gsteps <= kmax && !events(k + 1, k + gsteps) && A == A0) {
        if (!graph.exec && !graph.failed) {
          DACP_HIP(ctx, hipStreamSynchronize(ctx->stream));  // the first steps set the kernels' attributes
          graph.capture(gsteps, [&](int64_t j, hipStream_t cs) {
            double *tc = (j % 2 == 0) ? B0 : A0;
            double *tn = (j % 2 == 0) ? A0 : B0;
            return launch_step(k + j, tc, tn, nullptr, cs);
          });
        }
        if (graph.exec) {
          DACP_HIP(ctx, hipGraphLaunch(graph.exec, ctx->stream));
          launches += gsteps;
          k += gsteps;  // an even count: A and B are back in their roles
          continue;
        }
      }
      DACP_HIP(ctx, launch_step(k, B, A, store_of(k + 1), ctx->stream));
      ++k;
      ++launches;
      std::swap(A, B);
      if (want(k)) DACP_TRY(visit(k, B, A));
      if (verbose() && k % report_every == 0) {
        (void)hipStreamSynchronize(ctx->stream);
        vlog("evolution: step %lld of %lld (fused)", static_cast<long long>(k), static_cast<long long>(kmax));
      }
    }
    if (graph.exec) DACP_HIP(ctx, hipStreamSynchronize(ctx->stream));  // before the graph is released
    return DACP_OK;
  }
  for (int64_t k = 1; k < kmax; ++k) {
    st = step<double>(ctx, h, gw, B, gw, A, gw, 2.0 * inv_e, nullptr, 0, 0.0, A, gw, -1.0, store_of(k + 1), ldst, 2);
    if (st) return st;
    ++launches;
    std::swap(A, B);
    if (want(k + 1)) DACP_TRY(visit(k + 1, B, A));
    if (verbose() && (k + 1) % report_every == 0) {
      (void)hipStreamSynchronize(ctx->stream);
      vlog("evolution: step %lld of %lld", static_cast<long long>(k + 1), static_cast<long long>(kmax));
    }
  }
  return DACP_OK;
}

dacp_status run_basis(dacp_ctx ctx, dacp_ham h, const dacp_basis_params *p, const double *psi_e, double *V,
                      int64_t ldv, int *m_out, EvolStats *stats, bool onchip = true) {
  const int64_t D = h->D;
  const int b = p->b, n = p->n;
  if (b < 1 || n < 1 || !(p->e_bound > 0.0) || !(p->a > 0.0) || p->a >= p->e_bound || !psi_e || !V)
    return set_err(ctx, DACP_E_INVALID, "basis: need b >= 1, n >= 1, 0 < a < e_bound, psi_e, V");
  const int m = b * (2 * n + 1);
  if (ldv < m) return set_err(ctx, DACP_E_INVALID, "basis: ldv < b (2n + 1)");
  const double a_r = p->a / p->e_bound;
  const std::vector<int64_t> ks = sample_orders(a_r, n);
  std::map<int64_t, int> panel_of;  // order k -> panel index
  for (int i = 0; i < n; ++i) {
    panel_of[ks[i] - 1] = 2 * i + 1;
    panel_of[ks[i]] = 2 * i + 2;
  }
  const int64_t kmax = ks.back();
  const int gt = (p->group > 0 && p->group < b) ? p->group : recurrence_group(ctx, h, b);
  if (onchip && onchip_fits(ctx, h, b, ldv, static_cast<double>(kmax))) {
    Timer tm(ctx);
    tm.start();
    DACP_TRY(onchip_evolve(ctx, h, p->e_bound, b, psi_e, ks, V, ldv, nullptr, nullptr, 0, "basis"));
    if (m_out) *m_out = m;
    if (stats) *stats = {kmax, 1, tm.stop_ms(), gt};
    return DACP_OK;
  }
  const ColGroups cg = column_groups(ctx, h, b, gt, 3, {8});
  DevBuf ba, bb, nrm, pbuf;
  DACP_HIP(ctx, ba.alloc(cg.elems(D) * sizeof(double)));
  DACP_HIP(ctx, bb.alloc(cg.elems(D) * sizeof(double)));
  DACP_HIP(ctx, pbuf.alloc(cg.elems(D) * sizeof(double)));
  DACP_HIP(ctx, nrm.alloc(static_cast<size_t>(n) * b * sizeof(double)));
  const double inv_e = 1.0 / p->e_bound;
  Timer tm(ctx);
  tm.start();
  int64_t launches = 0;
  for (int g0 = 0; g0 < b; g0 += cg.cols(g0)) {
    const int nc = cg.cols(g0), gw = cg.width(g0), groups = cg.groups(g0);
    double *A = ba.as<double>(), *B = bb.as<double>();
    DACP_HIP(ctx, dacp::launch_split_cols(psi_e + g0, b, nc, A, D, gw, groups, ctx->stream));
    DACP_HIP(ctx, dacp::launch_copy_cols(psi_e + g0, b, V + g0, ldv, D, nc, ctx->stream));
    auto store_of = [&](int64_t k) -> double * {
      auto it = panel_of.find(k);
      return it == panel_of.end() ? nullptr : V + static_cast<int64_t>(it->second) * b + g0;
    };
    // whether a sample falls on T_k1 .. T_k2
    auto panel_in = [&](int64_t k1, int64_t k2) {
      auto it = panel_of.lower_bound(k1);
      return it != panel_of.end() && it->first <= k2;
    };
    dacp_status st = evolve_group(
        ctx, h, inv_e, kmax, gw, groups, nc, A, B, pbuf.as<double>(), store_of, ldv, [](int64_t) { return false; },
        [](int64_t, const double *, const double *) { return DACP_OK; }, panel_in, launches);
    if (st) return st;
  }
  const double evol_ms = tm.stop_ms();
  // |T_k(G)| <= 1 for e_bound >= ||H||: every stored T_{k_m} column must keep norm <= ||psi_E column||.
  std::vector<double> n0(b), nk(static_cast<size_t>(n) * b);
  dacp_status st = coldots_host(ctx, psi_e, b, psi_e, b, DACP_F64, D, b, n0.data());
  if (st) return st;
  for (int i = 0; i < n; ++i) {
    st = coldots_dev(ctx, V + static_cast<int64_t>(2 * i + 2) * b, ldv, V + static_cast<int64_t>(2 * i + 2) * b, ldv,
                     DACP_F64, D, b, nrm.as<double>() + static_cast<size_t>(i) * b);
    if (st) return st;
  }
  DACP_TRY(to_host(ctx, nk.data(), nrm.p, sizeof(double) * nk.size()));
  DACP_HIP(ctx, hipStreamSynchronize(ctx->stream));
  for (int i = 0; i < n; ++i)
    for (int j = 0; j < b; ++j) {
      const double v = nk[static_cast<size_t>(i) * b + j];
      if (!std::isfinite(v)) return set_err(ctx, DACP_E_NUMERIC, "basis: non-finite evolved state");
      if (v > n0[j] * (1.0 + 2e-6))
        return set_err(ctx, DACP_E_BOUNDS, "basis: |T_k(H/e_bound)| grew above 1; e_bound is below ||H||");
    }
  if (m_out) *m_out = m;
  if (stats) {
    stats->steps = kmax;
    stats->launches = launches;
    stats->kernel_ms = evol_ms;
    stats->group = gt;
  }
  return DACP_OK;
}

// ------------------------------------------------------------- projection
// K splits of the projection's small form (1: the shape does not take it): when the upper
// triangle of the m x m output has fewer 128 x 128 tiles than the GPU has compute units, K = D is
// split over up to 64 ranges of at least 1024 rows each.
int64_t project_small_splits(dacp_ctx ctx, int64_t D, int m) {
  const int64_t t = (m + 127) / 128, tu = t * (t + 1) / 2;
  if (!ctx->project_splitk || tu >= ctx->num_cus) return 1;
  return dacp::gemm_splits(m, m, D, 1, ctx->num_cus, 1024, 64);
}

// One product of the small form, queued on the context's stream without waiting: part 1 is
// S = V^T V, part 2 is P = V^T (H V).  Upper-triangle tiles with split K, then mirrored.  The
// scratch buffers are released on return; only stream-ordered reuse makes that safe before the
// kernels finish (the block cache of an AllocStream scope, or hipFree's device synchronisation).
dacp_status project_small(dacp_ctx ctx, dacp_ham h, int m, const double *V, int64_t ldv, double *out, int64_t ld,
                          int part) {
  const int64_t D = h->D;
  hipStream_t s = ctx->stream;
  const int sp = static_cast<int>(project_small_splits(ctx, D, m));
  DevBuf work, wall;
  DACP_HIP(ctx, work.alloc(static_cast<size_t>(sp) * m * m * sizeof(double)));
  const double *B = V;
  int64_t ldb = ldv;
  if (part == 2) {
    DACP_HIP(ctx, wall.alloc(static_cast<size_t>(D) * m * sizeof(double)));
    double *W = wall.as<double>();
    for (int s0 = 0; s0 < m; s0 += 64) {
      const int bw = std::min(64, m - s0);
      dacp_status st = step<double>(ctx, h, bw, V + s0, ldv, W + s0, m, 1.0);
      if (st) return st;
    }
    B = W;
    ldb = m;
  }
  DACP_HIP(ctx, dacp::launch_dgemm_splitk(1, 0, m, m, D, 1.0, V, ldv, B, ldb, 0.0, out, ld, 1, sp, work.as<double>(), s));
  DACP_HIP(ctx, dacp::launch_mirror_upper(out, m, ld, s));
  return DACP_OK;
}

// ------------------------------------------------------------- moment mode
// Moment mode (App. C, Eq. shift): the panels T_x(G) psi_E are never stored.  S and P follow from
// the b x b moments mu_k = psi_E^T T_k(G) psi_E and nu_k = psi_E^T G T_k(G) psi_E through
// T_x T_y = (T_{x+y} + T_{|x-y|}) / 2 and H = e_bound G:
//   S block (p, q) = (mu_{x+y} + mu_{|x-y|}) / 2,  P block (p, q) = e_bound (nu_{x+y} + nu_{|x-y|}) / 2.
// The samples sit on the uniform grid k_m = m Delta, Delta = 2 floor(pi / (2 a_r)), so that the
// orders x + y and |x - y| are recorded during an evolution to 2 k_n.  P is taken from nu rather
// than from mu one order off (G T_k = (T_{k+1} + T_{k-1}) / 2): the window's states have |G| <= a_r,
// so P is a_r times smaller than the moments, and differences of neighbouring mu would lose that
// factor of the recurrence's rounding.
struct MomentPlan {
  int64_t delta = 0;
  std::vector<int64_t> orders;  // panel orders: 0, k_1 - 1, k_1, ..., k_n - 1, k_n
};

MomentPlan moment_plan(double a_r, int n) {
  MomentPlan mp;
  mp.delta = std::max<int64_t>(2, 2 * static_cast<int64_t>(std::floor(M_PI / (2.0 * a_r))));
  mp.orders.push_back(0);
  for (int j = 1; j <= n; ++j) {
    mp.orders.push_back(j * mp.delta - 1);
    mp.orders.push_back(j * mp.delta);
  }
  return mp;
}

// Slot of every order x + y and |x - y| over the panel orders (-1 elsewhere, k = 0 .. 2 k_n), in
// order of first appearance; nslot gets the count.
std::vector<int> moment_slots(const std::vector<int64_t> &orders, int &nslot) {
  std::vector<int> slot_of(static_cast<size_t>(2 * orders.back()) + 1, -1);
  nslot = 0;
  for (int64_t x : orders)
    for (int64_t y : orders)
      for (int64_t k : {x + y, x >= y ? x - y : y - x})
        if (slot_of[k] < 0) slot_of[k] = nslot++;
  return slot_of;
}

// Columns of a D-row staging block, into z: `want`, or as many as a quarter of the free memory takes past
// 4 GiB, halved down to `least` until the allocation succeeds; 0 and no block when not even that does.
int staging_cols(int64_t D, int want, int least, DevBuf &z) {
  const size_t col = static_cast<size_t>(D) * sizeof(double);
  if (want > least && col * want > (size_t(4) << 30)) {
    size_t free_b = 0, total_b = 0;
    if (hipMemGetInfo(&free_b, &total_b) != hipSuccess) free_b = 0;
    want = std::max<int>(least, static_cast<int>(std::min<size_t>(want, free_b / 4 / col)));
  }
  while (z.alloc(col * want) != hipSuccess) {
    (void)hipGetLastError();
    if (want <= least) return 0;
    want = std::max(least, want / 2);
  }
  return want;
}

// Moment mode, first pass: filter output psi_e (D x b) -> S and P (device m x m, row stride ld),
// m = b (2n + 1).  Returns DACP_E_BOUNDS when |T_{k_m}(G) psi_j| exceeds |psi_j| (E_b < ||H||).
dacp_status run_moment_basis(dacp_ctx ctx, dacp_ham h, const dacp_basis_params *p, const double *psi_e, double *S,
                             double *P, int64_t ld, int *m_out, EvolStats *stats) {
  const int64_t D = h->D;
  const int b = p->b, n = p->n;
  if (b < 1 || b > 128 || n < 1 || !(p->e_bound > 0.0) || !(p->a > 0.0) || p->a >= p->e_bound || !psi_e || !S || !P)
    return set_err(ctx, DACP_E_INVALID, "basis_moments: need 1 <= b <= 128, n >= 1, 0 < a < e_bound, psi_e, S, P");
  const int m = b * (2 * n + 1);
  if (ld < m) return set_err(ctx, DACP_E_INVALID, "basis_moments: ld < b (2n + 1)");
  const MomentPlan mp = moment_plan(p->a / p->e_bound, n);
  const int64_t kmax = 2 * mp.orders.back();
  int nslot = 0;
  const std::vector<int> slot_of = moment_slots(mp.orders, nslot);
  const int g = (p->group > 0 && p->group < b) ? p->group : recurrence_group(ctx, h, b);
  const ColGroups cg = column_groups(ctx, h, b, g, 3, {8});
  const double inv_e = 1.0 / p->e_bound;
  // The recorded T_k are staged side by side, up to kz columns, and multiplied by [psi_E | G psi_E]^T
  // in one GEMM that gives mu and nu of them all: the left factor is read once for several orders.
  // (One 8-column group and factor at a time, on the vector ALU, a 2^16 x 32 order took 630 us.)
  // This is the mode for states too long to store a basis, so what it holds gives way to the memory
  // there is: the staged columns shrink to one launch's, then the products read T_k where it lies, and
  // psi_E is read from the caller's block.
  const int nc_max = std::min(b, cg.g * cg.per);
  DevBuf ba, bb, pbuf, left, mu, nu, zb, prod, work, didx, dord;
  DACP_HIP(ctx, ba.alloc(cg.elems(D) * sizeof(double)));
  DACP_HIP(ctx, bb.alloc(cg.elems(D) * sizeof(double)));
  DACP_HIP(ctx, pbuf.alloc(cg.elems(D) * sizeof(double)));
  DACP_HIP(ctx, mu.alloc(static_cast<size_t>(nslot) * b * b * sizeof(double)));
  DACP_HIP(ctx, nu.alloc(static_cast<size_t>(nslot) * b * b * sizeof(double)));
  const bool joined = left.alloc(static_cast<size_t>(D) * 2 * b * sizeof(double)) == hipSuccess;
  if (!joined) {
    (void)hipGetLastError();
    DACP_HIP(ctx, left.alloc(static_cast<size_t>(D) * b * sizeof(double)));
  }
  const int kz = staging_cols(D, std::max(256, nc_max), nc_max, zb);
  // rows and columns of one product: both factors or one, the staged columns or a group of T_k
  const int pm = joined ? 2 * b : b, pn = std::max(kz, cg.g);
  DACP_HIP(ctx, prod.alloc(static_cast<size_t>(pm) * pn * sizeof(double)));
  int sp = dacp::gemm_splits(pm, pn, D, 0, ctx->num_cus, 512, 128);
  if (sp > 1 && work.alloc(static_cast<size_t>(sp) * pm * pn * sizeof(double)) != hipSuccess) {
    (void)hipGetLastError();
    sp = 1;
  }
  double *const X = left.as<double>();
  double *const gpsi = joined ? X + b : X;
  const int64_t ldg = joined ? 2 * b : b;
  if (joined) DACP_HIP(ctx, dacp::launch_copy_cols(psi_e, b, X, 2 * b, D, b, ctx->stream));
  for (int c0 = 0; c0 < b; c0 += 64)
    DACP_TRY(step<double>(ctx, h, std::min(64, b - c0), psi_e + c0, b, gpsi + c0, ldg, inv_e));
  // moments of the w columns of Z (row stride ldz), a block of nc for each order of `at`, into columns
  // c0 .. c0 + nc - 1 of those orders' slots
  auto products = [&](const double *Z, int64_t ldz, int nc, const std::vector<int64_t> &at, int c0) -> dacp_status {
    const int w = static_cast<int>(at.size()) * nc;
    for (int f = 0; f < (joined ? 1 : 2); ++f) {
      const double *F = joined ? X : f ? gpsi : psi_e;
      if (sp > 1)
        DACP_HIP(ctx, dacp::launch_dgemm_splitk(1, 0, pm, w, D, 1.0, F, pm, Z, ldz, 0.0, prod.as<double>(), w, 0, sp,
                                                work.as<double>(), ctx->stream));
      else
        DACP_HIP(ctx, dacp::launch_dgemm(1, 0, pm, w, D, 1.0, F, pm, Z, ldz, 0.0, prod.as<double>(), w, 0, ctx->stream));
      for (size_t i = 0; i < at.size(); ++i)
        for (int q = f; q < (joined ? 2 : f + 1); ++q) {
          const double *src = prod.as<double>() + static_cast<int64_t>(i) * nc + (joined ? q : 0) * static_cast<int64_t>(b) * w;
          double *dst = (q ? nu : mu).as<double>() + static_cast<int64_t>(slot_of[at[i]]) * b * b + c0;
          DACP_HIP(ctx, dacp::launch_copy_cols(src, w, dst, b, b, nc, ctx->stream));
        }
    }
    return DACP_OK;
  };
  Timer tm(ctx);
  tm.start();
  int64_t launches = 0;
  for (int g0 = 0; g0 < b; g0 += cg.cols(g0)) {
    const int nc = cg.cols(g0), gw = cg.width(g0), groups = cg.groups(g0);
    double *A = ba.as<double>(), *B = bb.as<double>();
    DACP_HIP(ctx, dacp::launch_split_cols(psi_e + g0, b, nc, A, D, gw, groups, ctx->stream));
    auto want = [&](int64_t k) { return k <= kmax && slot_of[k] >= 0; };
    // mu_k[:, g0 .. g0 + nc) = psi_E^T (T_k psi_E)[:, these columns], nu_k likewise with (G psi_E)^T
    std::vector<int64_t> staged;  // orders of the staged blocks of nc columns
    auto flush = [&]() -> dacp_status {
      if (!staged.empty()) DACP_TRY(products(zb.as<double>(), kz, nc, staged, g0));
      staged.clear();
      return DACP_OK;
    };
    auto visit = [&](int64_t k, const double *tk, const double *) -> dacp_status {
      if (kz == 0) {
        for (int y = 0; y < groups; ++y)
          DACP_TRY(products(tk + y * D * gw, gw, std::min(gw, nc - y * gw), {k}, g0 + y * gw));
        return DACP_OK;
      }
      DACP_HIP(ctx, dacp::launch_join_cols(tk, D, gw, groups, zb.as<double>() + staged.size() * nc, kz, nc, ctx->stream));
      staged.push_back(k);
      if (static_cast<int>(staged.size() + 1) * nc > kz) return flush();
      return DACP_OK;
    };
    auto events = [&](int64_t k1, int64_t k2) {
      for (int64_t k = k1; k <= k2 && k <= kmax; ++k)
        if (slot_of[k] >= 0) return true;
      return false;
    };
    dacp_status st = evolve_group(
        ctx, h, inv_e, kmax, gw, groups, nc, A, B, pbuf.as<double>(), [](int64_t) -> double * { return nullptr; }, 0,
        want, visit, events, launches);
    if (st) return st;
    DACP_TRY(flush());
  }
  const double evol_ms = tm.stop_ms();
  // |T_k(G)| <= 1 for e_bound >= ||H||: |T_{k_j} psi|^2 = (mu_{2 k_j} + mu_0) / 2 on the diagonal
  std::vector<double> muh(static_cast<size_t>(nslot) * b * b);
  DACP_TRY(to_host(ctx, muh.data(), mu.p, muh.size() * sizeof(double)));
  auto mu_at = [&](int64_t k, int i, int j) { return muh[(static_cast<size_t>(slot_of[k]) * b + i) * b + j]; };
  for (int j = 1; j <= n; ++j)
    for (int c = 0; c < b; ++c) {
      const double n0 = mu_at(0, c, c);
      const double nk = 0.5 * (mu_at(2 * j * mp.delta, c, c) + n0);
      if (!std::isfinite(nk) || !std::isfinite(n0)) return set_err(ctx, DACP_E_NUMERIC, "basis_moments: non-finite moment");
      if (nk > n0 * (1.0 + 4e-6))
        return set_err(ctx, DACP_E_BOUNDS, "basis_moments: |T_k(H/e_bound)| grew above 1; e_bound is below ||H||");
    }
  DACP_HIP(ctx, didx.alloc(slot_of.size() * sizeof(int)));
  DACP_HIP(ctx, dord.alloc(mp.orders.size() * sizeof(int64_t)));
  DACP_TRY(to_device(ctx, didx.p, slot_of.data(), slot_of.size() * sizeof(int)));
  DACP_TRY(to_device(ctx, dord.p, mp.orders.data(), mp.orders.size() * sizeof(int64_t)));
  const int npan = static_cast<int>(mp.orders.size());
  DACP_HIP(ctx, dacp::launch_gram_assemble(mu.as<double>(), didx.as<int>(), dord.as<int64_t>(), b, npan, 1.0, S, ld,
                                           ctx->stream));
  DACP_HIP(ctx, dacp::launch_gram_assemble(nu.as<double>(), didx.as<int>(), dord.as<int64_t>(), b, npan, p->e_bound, P,
                                           ld, ctx->stream));
  // the moments are symmetric only up to rounding: take the symmetric parts
  DACP_HIP(ctx, dacp::launch_symmetrize(S, m, ld, ctx->stream));
  DACP_HIP(ctx, dacp::launch_symmetrize(P, m, ld, ctx->stream));
  DACP_HIP(ctx, hipStreamSynchronize(ctx->stream));
  if (m_out) *m_out = m;
  if (stats) {
    stats->steps = kmax;
    stats->launches = launches;
    stats->kernel_ms = evol_ms;
    stats->group = g;
  }
  return DACP_OK;
}

// Moment mode, second pass: the Ritz vectors of nc candidates, Phi = A Bc (D x nc, row stride nc),
// accumulated during an evolution to k_n without storing A.  bsel (device nc x m, row stride m):
// row c is column c of B.  Panels are staged a few hundred columns at a time, then added with one
// GEMM Phi += Z W^T, W (nc x K) the matching columns of bsel.
dacp_status moment_ritz_vectors(dacp_ctx ctx, dacp_ham h, const dacp_basis_params *p, const double *psi_e,
                                const double *bsel, int nc, double *Phi, EvolStats *stats) {
  const int64_t D = h->D;
  const int b = p->b, n = p->n;
  const int m = b * (2 * n + 1);
  const MomentPlan mp = moment_plan(p->a / p->e_bound, n);
  std::map<int64_t, int> panel_of;  // panel order -> panel index
  for (size_t q = 0; q < mp.orders.size(); ++q) panel_of[mp.orders[q]] = static_cast<int>(q);
  const int64_t kmax = mp.orders.back();
  const int g = (p->group > 0 && p->group < b) ? p->group : recurrence_group(ctx, h, b);
  const ColGroups cg = column_groups(ctx, h, b, g, 3, {8});
  const double inv_e = 1.0 / p->e_bound;
  DevBuf ba, bb, pbuf, zb, wb, dcols;
  DACP_HIP(ctx, ba.alloc(cg.elems(D) * sizeof(double)));
  DACP_HIP(ctx, bb.alloc(cg.elems(D) * sizeof(double)));
  DACP_HIP(ctx, pbuf.alloc(cg.elems(D) * sizeof(double)));
  // staged columns: 32 groups of the requested width, at least one of the launch's
  const int kz = staging_cols(D, std::max(32 * g, cg.g), cg.g, zb);
  if (kz == 0) return set_err(ctx, DACP_E_NOMEM, "moment mode: staging block");
  DACP_HIP(ctx, wb.alloc(static_cast<size_t>(nc) * kz * sizeof(double)));
  DACP_HIP(ctx, dcols.alloc(static_cast<size_t>(kz) * sizeof(int)));
  DACP_HIP(ctx, hipMemsetAsync(Phi, 0, static_cast<size_t>(D) * nc * sizeof(double), ctx->stream));
  std::vector<int> cols;  // columns of bsel (index into m) of the staged Z columns
  int64_t launches = 0;
  Timer tm(ctx);
  tm.start();
  auto flush = [&]() -> dacp_status {
    if (cols.empty()) return DACP_OK;
    const int K = static_cast<int>(cols.size());
    DACP_TRY(to_device(ctx, dcols.p, cols.data(), cols.size() * sizeof(int)));
    DACP_HIP(ctx, dacp::launch_gather_cols(bsel, m, dcols.as<int>(), nullptr, nc, K, wb.as<double>(), K, ctx->stream));
    DACP_HIP(ctx, dacp::launch_dgemm(0, 1, D, nc, K, 1.0, zb.as<double>(), kz, wb.as<double>(), K, 1.0, Phi, nc, 0,
                                     ctx->stream));
    cols.clear();  // the next copies into Z and dcols are queued behind this GEMM on the same stream
    return DACP_OK;
  };
  for (int g0 = 0; g0 < b; g0 += cg.cols(g0)) {
    const int nc = cg.cols(g0), gw = cg.width(g0), groups = cg.groups(g0);
    double *A = ba.as<double>(), *B = bb.as<double>();
    DACP_HIP(ctx, dacp::launch_split_cols(psi_e + g0, b, nc, A, D, gw, groups, ctx->stream));
    auto want = [&](int64_t k) { return panel_of.count(k) > 0; };
    auto visit = [&](int64_t k, const double *tk, const double *) -> dacp_status {
      const int pidx = panel_of[k];
      for (int y = 0; y < groups; ++y) {
        const int yc = std::min(gw, nc - y * gw);
        if (static_cast<int>(cols.size()) + yc > kz) DACP_TRY(flush());
        const int slot0 = static_cast<int>(cols.size());
        DACP_HIP(ctx, dacp::launch_copy_cols(tk + y * D * gw, gw, zb.as<double>() + slot0, kz, D, yc, ctx->stream));
        for (int c = 0; c < yc; ++c) cols.push_back(pidx * b + g0 + y * gw + c);
      }
      return DACP_OK;
    };
    auto events = [&](int64_t k1, int64_t k2) {
      auto it = panel_of.lower_bound(k1);
      return it != panel_of.end() && it->first <= k2;
    };
    dacp_status st = evolve_group(
        ctx, h, inv_e, kmax, gw, groups, nc, A, B, pbuf.as<double>(), [](int64_t) -> double * { return nullptr; }, 0,
        want, visit, events, launches);
    if (st) return st;
  }
  DACP_TRY(flush());
  if (stats) {
    stats->steps += kmax;
    stats->launches += launches;
    stats->kernel_ms += tm.stop_ms();
  }
  return DACP_OK;
}

// Stored basis with moment projection (App. C, Eq. shift): the panels of the uniform grid are
// stored in V as by the evolution basis, and S and P are assembled from b x b moments, but the moments
// come from Gram products of a few anchor panels with V instead of an evolution to 2 k_n.  For
// an anchor T_A psi and a panel T_x psi (G = H / e_bound),
//   (T_A psi)^T (T_x psi)   = (mu_{A+x} + mu_{|A-x|}) / 2,  mu_k = psi^T T_k(G) psi,
//   (H T_A psi)^T (T_x psi) = e_bound (nu_{A+x} + nu_{|A-x|}) / 2,  nu_k = psi^T G T_k(G) psi,
// so a moment follows from one such block and the moment at the other order.  The anchors are the
// orders 0, 1, 2 and k_n - 2 .. k_n + 1 (k_n the last sample): those next to 0 give every moment up to
// about k_n, those next to k_n the ones beyond.  Then S block (p, q) = (mu_{x+y} + mu_{|x-y|}) / 2 and
// P block (p, q) = e_bound (nu_{x+y} + nu_{|x-y|}) / 2.  P is taken from nu rather than from mu one
// order off (T_1 T_k = (T_{k+1} + T_{k-1}) / 2): the window's states have |G| <= a_r, so P is a_r
// times smaller than the moments, and differences of neighbouring mu would lose that factor of the
// recurrence's rounding.  The Gram products cost 2 D (14 b) m flops against 2 D m^2 for V^T V and
// V^T (H V).
// S and P (device m x m, row stride ld) of the panels of orders `orders` stored in V (device D x m,
// row stride ldv) from the anchors: abuf (device D x 2 na b, row stride 2 na b) holds T_A psi of
// anchor i = 0 .. na-1 in columns [i b, i b + b); its right half receives their images under H.
// gram_ms (may be null) gets the wall time of the whole step.
dacp_status anchor_projection(dacp_ctx ctx, dacp_ham h, const std::vector<int64_t> &orders,
                              const std::vector<int64_t> &anchors, double *abuf, const double *V, int64_t ldv, int b,
                              double e_bound, double *S, double *P, int64_t ld, double *gram_ms) {
  const int64_t D = h->D;
  hipStream_t s = ctx->stream;
  const int npan = static_cast<int>(orders.size());
  const int m = b * npan;
  const int na = static_cast<int>(anchors.size());
  const int ma = na * b;
  // images of the anchors under H, beside them
  const double tg0 = now_ms();
  for (int c0 = 0; c0 < ma; c0 += 64)
    DACP_TRY(step<double>(ctx, h, std::min(64, ma - c0), abuf + c0, 2 * ma, abuf + ma + c0, 2 * ma, 1.0));
  // Gram of the anchors and their images with the panels, (2 na b) x m: block (i, q) =
  // (T_{anchors[i]} psi)^T (T_{orders[q]} psi), block (na + i, q) = (H T_{anchors[i]} psi)^T (T_{orders[q]} psi)
  const int mg = 2 * ma;
  DevBuf gd;
  DACP_HIP(ctx, gd.alloc(static_cast<size_t>(mg) * m * sizeof(double)));
  {
    DevBuf work;
    int sp = dacp::gemm_splits(mg, m, D, 0, ctx->num_cus, 1024, 64);
    if (sp > 1 && work.alloc(static_cast<size_t>(sp) * mg * m * sizeof(double)) != hipSuccess) {
      (void)hipGetLastError();
      sp = 1;
    }
    if (sp > 1) {
      DACP_HIP(ctx, dacp::launch_dgemm_splitk(1, 0, mg, m, D, 1.0, abuf, mg, V, ldv, 0.0, gd.as<double>(), m, 0, sp,
                                              work.as<double>(), s));
    } else {
      DACP_HIP(ctx, dacp::launch_dgemm(1, 0, mg, m, D, 1.0, abuf, mg, V, ldv, 0.0, gd.as<double>(), m, 0,
                                       s));
    }
  }
  // the chain of Gram blocks that gives every moment S and P read (host rule, integers only)
  const dacp::rules::MomentChain ch = dacp::rules::moment_chain(orders, anchors);
  if (ch.missing >= 0)
    return set_err(ctx, DACP_E_INVALID, "basis_stored_moments: moment " + std::to_string(ch.missing) + " not reachable");
  const std::vector<int> &table = ch.table, &block_of = ch.block_of;
  const int nc = static_cast<int>(ch.order.size());
  // the moments on the device: mu from the anchor rows, nu from the image rows scaled by 1 / e_bound
  const size_t bb2 = static_cast<size_t>(b) * b;
  DevBuf mom, drules, dblk, dord, dbad;
  DACP_HIP(ctx, mom.alloc(2 * static_cast<size_t>(nc) * bb2 * sizeof(double)));
  DACP_HIP(ctx, drules.alloc(table.size() * sizeof(int)));
  DACP_HIP(ctx, dblk.alloc(block_of.size() * sizeof(int)));
  DACP_HIP(ctx, dord.alloc(orders.size() * sizeof(int64_t)));
  DACP_HIP(ctx, dbad.alloc(sizeof(int)));
  DACP_TRY(to_device(ctx, drules.p, table.data(), table.size() * sizeof(int)));
  DACP_TRY(to_device(ctx, dblk.p, block_of.data(), block_of.size() * sizeof(int)));
  DACP_TRY(to_device(ctx, dord.p, orders.data(), orders.size() * sizeof(int64_t)));
  const int zero = 0;
  DACP_TRY(to_device(ctx, dbad.p, &zero, sizeof(int)));
  DACP_HIP(ctx, dacp::launch_moment_chain(gd.as<double>(), m, b, na, drules.as<int>(), nc, 1.0, 1.0 / e_bound,
                                          mom.as<double>(), dbad.as<int>(), s));
  int bad = 0;
  DACP_TRY(to_host(ctx, &bad, dbad.p, sizeof(int)));
  if (bad) return set_err(ctx, DACP_E_NUMERIC, "basis_stored_moments: non-finite moment");
  const double *mu = mom.as<double>(), *nu = mu + static_cast<size_t>(nc) * bb2;
  DACP_HIP(ctx, dacp::launch_gram_assemble(mu, dblk.as<int>(), dord.as<int64_t>(), b, npan, 1.0, S, ld, s));
  DACP_HIP(ctx, dacp::launch_gram_assemble(nu, dblk.as<int>(), dord.as<int64_t>(), b, npan, e_bound, P, ld, s));
  DACP_HIP(ctx, dacp::launch_symmetrize(S, m, ld, s));
  DACP_HIP(ctx, dacp::launch_symmetrize(P, m, ld, s));
  DACP_HIP(ctx, hipStreamSynchronize(s));
  if (gram_ms) *gram_ms = now_ms() - tg0;
  return DACP_OK;
}

dacp_status run_stored_moment_basis(dacp_ctx ctx, dacp_ham h, const dacp_basis_params *p, const double *psi_e,
                                    double *V, int64_t ldv, double *S, double *P, int64_t ld, int *m_out,
                                    EvolStats *stats, double *gram_ms) {
  const int64_t D = h->D;
  const int b = p->b, n = p->n;
  if (b < 1 || b > 128 || n < 1 || !(p->e_bound > 0.0) || !(p->a > 0.0) || p->a >= p->e_bound || !psi_e || !V ||
      !S || !P)
    return set_err(ctx, DACP_E_INVALID,
                   "basis_stored_moments: need 1 <= b <= 128, n >= 1, 0 < a < e_bound, psi_e, V, S, P");
  const int m = b * (2 * n + 1);
  if (ldv < m || ld < m) return set_err(ctx, DACP_E_INVALID, "basis_stored_moments: ldv or ld < b (2n + 1)");
  hipStream_t s = ctx->stream;
  const MomentPlan mp = moment_plan(p->a / p->e_bound, n);
  const int npan = static_cast<int>(mp.orders.size());
  std::map<int64_t, int> panel_of;  // panel order -> panel index
  for (int q = 0; q < npan; ++q) panel_of[mp.orders[q]] = q;
  const int64_t kn = mp.orders.back();
  const std::vector<int64_t> anchors = anchor_orders(kn);
  std::map<int64_t, int> anchor_of;  // anchor order -> anchor slot
  for (size_t i = 0; i < anchors.size(); ++i) anchor_of[anchors[i]] = static_cast<int>(i);
  const int na = static_cast<int>(anchors.size());
  const int ma = na * b;  // anchor block width
  const int gt = (p->group > 0 && p->group < b) ? p->group : recurrence_group(ctx, h, b);
  if (onchip_fits(ctx, h, b, std::max<int64_t>(ldv, 2 * ma), static_cast<double>(kn + 1))) {
    std::vector<int64_t> ks;
    for (int j = 1; j <= n; ++j) ks.push_back(mp.orders[2 * j]);
    DevBuf abuf;
    DACP_HIP(ctx, abuf.alloc(static_cast<size_t>(D) * 2 * ma * sizeof(double)));
    Timer tm(ctx);
    tm.start();
    DACP_TRY(onchip_evolve(ctx, h, p->e_bound, b, psi_e, ks, V, ldv, &anchors, abuf.as<double>(), 2 * ma,
                           "basis_stored_moments"));
    const double evol_ms = tm.stop_ms();
    DACP_TRY(anchor_projection(ctx, h, mp.orders, anchors, abuf.as<double>(), V, ldv, b, p->e_bound, S, P, ld, gram_ms));
    if (m_out) *m_out = m;
    if (stats) *stats = {kn + 1, 1, evol_ms, gt};
    return DACP_OK;
  }
  const ColGroups cg = column_groups(ctx, h, b, gt, 3, {8});
  const double inv_e = 1.0 / p->e_bound;
  DevBuf ba, bb, pbuf, abuf, nrm;
  DACP_HIP(ctx, ba.alloc(cg.elems(D) * sizeof(double)));
  DACP_HIP(ctx, bb.alloc(cg.elems(D) * sizeof(double)));
  DACP_HIP(ctx, pbuf.alloc(cg.elems(D) * sizeof(double)));
  DACP_HIP(ctx, abuf.alloc(static_cast<size_t>(D) * 2 * ma * sizeof(double)));  // anchors | their H images
  DACP_HIP(ctx, nrm.alloc(static_cast<size_t>(n) * b * sizeof(double)));
  Timer tm(ctx);
  tm.start();
  int64_t launches = 0;
  for (int g0 = 0; g0 < b; g0 += cg.cols(g0)) {
    const int nc = cg.cols(g0), gw = cg.width(g0), groups = cg.groups(g0);
    double *A = ba.as<double>(), *B = bb.as<double>();
    DACP_HIP(ctx, dacp::launch_split_cols(psi_e + g0, b, nc, A, D, gw, groups, s));
    DACP_HIP(ctx, dacp::launch_copy_cols(psi_e + g0, b, V + g0, ldv, D, nc, s));
    auto store_of = [&](int64_t k) -> double * {
      auto it = panel_of.find(k);
      return (k == 0 || it == panel_of.end()) ? nullptr : V + static_cast<int64_t>(it->second) * b + g0;
    };
    auto want = [&](int64_t k) { return anchor_of.count(k) > 0; };
    auto visit = [&](int64_t k, const double *tk, const double *) -> dacp_status {
      DACP_HIP(ctx, dacp::launch_join_cols(tk, D, gw, groups,
                                           abuf.as<double>() + static_cast<int64_t>(anchor_of[k]) * b + g0, 2 * ma, nc,
                                           s));
      return DACP_OK;
    };
    auto events = [&](int64_t k1, int64_t k2) {
      auto it = panel_of.lower_bound(k1);
      if (it != panel_of.end() && it->first <= k2) return true;
      auto ia = anchor_of.lower_bound(k1);
      return ia != anchor_of.end() && ia->first <= k2;
    };
    dacp_status st =
        evolve_group(ctx, h, inv_e, kn + 1, gw, groups, nc, A, B, pbuf.as<double>(), store_of, ldv, want, visit, events,
                     launches);
    if (st) return st;
  }
  const double evol_ms = tm.stop_ms();
  // |T_k(G)| <= 1 for e_bound >= ||H||: every stored T_{k_j} column must keep norm <= ||psi_E column||
  std::vector<double> n0(b), nk(static_cast<size_t>(n) * b);
  DACP_TRY(coldots_host(ctx, psi_e, b, psi_e, b, DACP_F64, D, b, n0.data()));
  for (int j = 1; j <= n; ++j)
    DACP_TRY(coldots_dev(ctx, V + static_cast<int64_t>(2 * j) * b, ldv, V + static_cast<int64_t>(2 * j) * b, ldv,
                         DACP_F64, D, b, nrm.as<double>() + static_cast<size_t>(j - 1) * b));
  DACP_TRY(to_host(ctx, nk.data(), nrm.p, sizeof(double) * nk.size()));
  DACP_HIP(ctx, hipStreamSynchronize(s));
  for (size_t i = 0; i < nk.size(); ++i) {
    if (!std::isfinite(nk[i])) return set_err(ctx, DACP_E_NUMERIC, "basis_stored_moments: non-finite evolved state");
    if (nk[i] > n0[i % b] * (1.0 + 2e-6))
      return set_err(ctx, DACP_E_BOUNDS, "basis_stored_moments: |T_k(H/e_bound)| grew above 1; e_bound is below ||H||");
  }
  DACP_TRY(anchor_projection(ctx, h, mp.orders, anchors, abuf.as<double>(), V, ldv, b, p->e_bound, S, P, ld, gram_ms));
  if (m_out) *m_out = m;
  if (stats) {
    stats->steps = kn + 1;
    stats->launches = launches;
    stats->kernel_ms = evol_ms;
    stats->group = gt;
  }
  return DACP_OK;
}

dacp_status run_project(dacp_ctx ctx, dacp_ham h, int m, const double *V, int64_t ldv, double *S, double *P,
                        int64_t ld) {
  const int64_t D = h->D;
  if (m < 1 || ldv < m || ld < m || !V || !S || !P) return set_err(ctx, DACP_E_INVALID, "project: bad sizes/pointers");
  hipStream_t s = ctx->stream;
  Timer ts(ctx);
  if (verbose()) ts.start();
  // Few output tiles against a long K (the small subspaces of batched realisations): both products
  // as upper-triangle tiles with K split over workgroup layers, then mirrored as below.
  if (project_small_splits(ctx, D, m) > 1) {
    DACP_TRY(project_small(ctx, h, m, V, ldv, S, ld, 1));
    DACP_TRY(project_small(ctx, h, m, V, ldv, P, ld, 2));
    if (verbose()) vlog("projection: S and P with split K (m = %d) %.1f ms", m, ts.stop_ms());
    DACP_HIP(ctx, hipStreamSynchronize(s));
    return DACP_OK;
  }
  // The large form: upper-triangle tiles, K split a few ways where that fills the last round of
  // workgroups better and the scratch fits.
  DevBuf split_work;
  int big_splits = ctx->project_splitk ? dacp::gemm_splits(m, m, D, 1, ctx->num_cus, 4096, 4) : 1;
  if (big_splits > 1 &&
      split_work.alloc(static_cast<size_t>(big_splits) * m * m * sizeof(double)) != hipSuccess)
    big_splits = 1;
  (void)hipGetLastError();
  auto gram_upper = [&](const double *B, int64_t ldb, double *C) -> hipError_t {
    return big_splits > 1 ? dacp::launch_dgemm_splitk(1, 0, m, m, D, 1.0, V, ldv, B, ldb, 0.0, C, ld, 1, big_splits,
                                                      split_work.as<double>(), s)
                          : dacp::launch_dgemm(1, 0, m, m, D, 1.0, V, ldv, B, ldb, 0.0, C, ld, 1, s);
  };
  DACP_HIP(ctx, gram_upper(V, ldv, S));
  DACP_HIP(ctx, dacp::launch_mirror_upper(S, m, ld, s));
  if (verbose()) {
    const double ms = ts.stop_ms();
    vlog("projection: S = V^T V (m = %d) %.1f ms, %.1f TFLOP/s (upper tiles)", m, ms,
         static_cast<double>(D) * m * (m + 128.0) / (ms * 1e-3) / 1e12);
    ts.start();
  }
  // With room for the whole block H V (D x m) beside V, P is one upper-triangle GEMM like S;
  // otherwise it is built in column chunks of 512 against the rows up to each chunk's end.
  {
    const size_t whole = static_cast<size_t>(D) * m * sizeof(double);
    size_t free_b = 0, total_b = 0;
    DevBuf wall;
    if (ctx->project_whole && hipMemGetInfo(&free_b, &total_b) == hipSuccess && free_b > whole + (size_t(4) << 30) &&
        wall.alloc(whole) == hipSuccess) {
      double *W = wall.as<double>();
      for (int s0 = 0; s0 < m; s0 += 64) {
        const int bw = std::min(64, m - s0);
        dacp_status st = step<double>(ctx, h, bw, V + s0, ldv, W + s0, m, 1.0);
        if (st) return st;
      }
      DACP_HIP(ctx, gram_upper(W, m, P));
      DACP_HIP(ctx, dacp::launch_mirror_upper(P, m, ld, s));
      if (verbose()) vlog("projection: P = V^T (H V) in one GEMM %.1f ms", ts.stop_ms());
      DACP_HIP(ctx, hipStreamSynchronize(s));
      return DACP_OK;
    }
    (void)hipGetLastError();  // a failed allocation here only selects the chunked form
  }
  split_work.release();  // S is queued, and the chunks' buffers come first
  const int cw = std::min(m, 512);
  DevBuf wbuf;
  DACP_HIP(ctx, wbuf.alloc(static_cast<size_t>(D) * cw * sizeof(double)));
  double *W = wbuf.as<double>();
  // The early chunks have few output tiles against a K of 2^L: split K to fill the GPU, if there is room.
  int max_splits = 64;
  auto splits_for = [&](int rows, int cols) {
    return dacp::gemm_splits(rows, cols, D, 0, ctx->num_cus, 1024, max_splits);
  };
  size_t work_elems = 0;
  for (int c0 = 0; c0 < m; c0 += cw) {
    const int c1 = std::min(m, c0 + cw);
    const int sp = splits_for(c1, c1 - c0);
    if (sp > 1) work_elems = std::max(work_elems, static_cast<size_t>(sp) * c1 * (c1 - c0));
  }
  DevBuf work;
  if (work_elems && work.alloc(work_elems * sizeof(double)) != hipSuccess) {
    (void)hipGetLastError();
    max_splits = 1;
  }
  for (int c0 = 0; c0 < m; c0 += cw) {
    const int c1 = std::min(m, c0 + cw);
    const int w = c1 - c0;
    for (int s0 = c0; s0 < c1; s0 += 64) {
      const int bw = std::min(64, c1 - s0);
      dacp_status st = step<double>(ctx, h, bw, V + s0, ldv, W + (s0 - c0), cw, 1.0);
      if (st) return st;
    }
    const int sp = splits_for(c1, w);
    if (sp > 1)
      DACP_HIP(ctx, dacp::launch_dgemm_splitk(1, 0, c1, w, D, 1.0, V, ldv, W, cw, 0.0, P + c0, ld, 0, sp,
                                              work.as<double>(), s));
    else
      DACP_HIP(ctx, dacp::launch_dgemm(1, 0, c1, w, D, 1.0, V, ldv, W, cw, 0.0, P + c0, ld, 0, s));
  }
  DACP_HIP(ctx, dacp::launch_mirror_upper(P, m, ld, s));
  if (verbose()) vlog("projection: P = V^T (H V) in chunks %.1f ms", ts.stop_ms());
  DACP_HIP(ctx, hipStreamSynchronize(s));
  return DACP_OK;
}

// ----------------------------------------------------- Rayleigh-Ritz (App. C)
// App. C after the eigen-decomposition of S (lam ascending, zs rows = eigenvectors): drop the
// eigenvalues at or below eps, U = V~ Lambda~^(-1/2) stored as the rows of uc (r x m), and
// H~ = U^T P U (r x r, symmetrised) in ht.
dacp_status rr_reduce(dacp_ctx ctx, int m, const std::vector<double> &lam, const double *zs, const double *P,
                      int64_t ld, double eps, DevBuf &uc, DevBuf &ht, int *r_out) {
  hipStream_t s = ctx->stream;
  int i0 = 0;
  while (i0 < m && !(lam[i0] > eps)) ++i0;
  const int r = m - i0;
  if (r == 0) return set_err(ctx, DACP_E_NUMERIC, "overlap matrix S has no eigenvalue above eps");
  std::vector<int> perm(r);
  std::vector<double> scale(r);
  for (int t = 0; t < r; ++t) {
    perm[t] = i0 + t;
    scale[t] = 1.0 / std::sqrt(lam[i0 + t]);
  }
  DevBuf dperm, dscale, t1;
  DACP_HIP(ctx, dperm.alloc(sizeof(int) * r));
  DACP_HIP(ctx, dscale.alloc(sizeof(double) * r));
  DACP_TRY(to_device(ctx, dperm.p, perm.data(), sizeof(int) * r));
  DACP_TRY(to_device(ctx, dscale.p, scale.data(), sizeof(double) * r));
  DACP_HIP(ctx, uc.alloc(static_cast<size_t>(r) * m * sizeof(double)));
  DACP_HIP(ctx, dacp::launch_gather_rows(zs, m, uc.as<double>(), m, dperm.as<int>(), dscale.as<double>(), r, m, s));
  // H~ = U^T P U with U = columns of Uc^T:  T1 = Uc P (r x m),  H~ = T1 Uc^T (r x r).
  DACP_HIP(ctx, t1.alloc(static_cast<size_t>(r) * m * sizeof(double)));
  DACP_HIP(ctx, dacp::launch_dgemm(0, 0, r, m, m, 1.0, uc.as<double>(), m, P, ld, 0.0, t1.as<double>(), m, 0, s));
  DACP_HIP(ctx, ht.alloc(static_cast<size_t>(r) * r * sizeof(double)));
  DACP_HIP(ctx, dacp::launch_dgemm(0, 1, r, r, m, 1.0, t1.as<double>(), m, uc.as<double>(), m, 0.0, ht.as<double>(), r,
                                   0, s));
  DACP_HIP(ctx, dacp::launch_symmetrize(ht.as<double>(), r, r, s));
  DACP_HIP(ctx, hipStreamSynchronize(s));  // dperm, dscale, t1 are released on return
  *r_out = r;
  return DACP_OK;
}

// App. C after the eigen-decomposition of H~ (theta ascending, yc rows = eigenvectors): the rows of
// B^T, Bc = Yc Uc (r x m), and a finiteness check of the Ritz values.
dacp_status rr_back(dacp_ctx ctx, int m, int r, const double *yc, const double *uc, const std::vector<double> &theta,
                    DevBuf *bc_out) {
  if (bc_out) {
    DACP_HIP(ctx, bc_out->alloc(static_cast<size_t>(r) * m * sizeof(double)));
    DACP_HIP(ctx, dacp::launch_dgemm(0, 0, r, m, r, 1.0, yc, r, uc, m, 0.0, bc_out->as<double>(), m, 0, ctx->stream));
    DACP_HIP(ctx, hipStreamSynchronize(ctx->stream));
  }
  for (double t : theta)
    if (!std::isfinite(t)) return set_err(ctx, DACP_E_NUMERIC, "non-finite Ritz value");
  return DACP_OK;
}

// A dense symmetric eigensolver (n, A device n x n destroyed, w host ascending, Zrows device or null).
typedef std::function<dacp_status(int, double *, double *, double *)> EigFn;

dacp_status run_rr(dacp_ctx ctx, int m, const double *S, const double *P, int64_t ld, double eps,
                   std::vector<double> &theta, DevBuf *bc_out, int *r_out, const EigFn *eig = nullptr) {
  auto solve = [&](int n, double *A, double *w, double *Z) -> dacp_status {
    return eig ? (*eig)(n, A, w, Z) : dacp::gpu_syev(ctx, n, A, n, w, Z);
  };
  hipStream_t s = ctx->stream;
  DevBuf awork, zs;
  DACP_HIP(ctx, awork.alloc(static_cast<size_t>(m) * m * sizeof(double)));
  DACP_HIP(ctx, zs.alloc(static_cast<size_t>(m) * m * sizeof(double)));
  DACP_HIP(ctx, dacp::launch_copy_cols(S, ld, awork.as<double>(), m, m, m, s));
  std::vector<double> lam(m);
  dacp_status st = solve(m, awork.as<double>(), lam.data(), zs.as<double>());
  if (st) return st;
  DevBuf uc, ht, yc;
  int r = 0;
  st = rr_reduce(ctx, m, lam, zs.as<double>(), P, ld, eps, uc, ht, &r);
  if (st) return st;
  zs.release();
  awork.release();
  theta.assign(r, 0.0);
  const bool want_b = bc_out != nullptr;
  if (want_b) DACP_HIP(ctx, yc.alloc(static_cast<size_t>(r) * r * sizeof(double)));
  st = solve(r, ht.as<double>(), theta.data(), want_b ? yc.as<double>() : nullptr);
  if (st) return st;
  st = rr_back(ctx, m, r, want_b ? yc.as<double>() : nullptr, uc.as<double>(), theta, bc_out);
  if (st) return st;
  if (r_out) *r_out = r;
  return DACP_OK;
}

// ---------------------------------------------------------- Lanczos bound
// E_b from the Lanczos tridiagonal (alpha, beta): the extreme Ritz values widened by their Ritz
// residuals |beta_k y_k|, times `safety`, clamped to sum |c| (reading of the Sec. III estimator).
dacp_status lanczos_bound(dacp_ctx ctx, const std::vector<double> &al, const std::vector<double> &be, double safety,
                          double sum_abs, double *e_bound, double *tmin, double *tmax) {
  const int k = static_cast<int>(al.size());
  if (k < 1 || be.size() != al.size()) return set_err(ctx, DACP_E_NUMERIC, "bound: empty Lanczos run");
  std::vector<double> th(k), Z(static_cast<size_t>(k) * k);
  if (!dacp::host_tridiag_eig(al.data(), be.data(), k, th.data(), Z.data()))
    return set_err(ctx, DACP_E_CONVERGENCE, "bound: tridiagonal eigensolver");
  const double bk = be.back();
  const double r_lo = std::fabs(bk * Z[static_cast<size_t>(k - 1) * k + 0]);
  const double r_hi = std::fabs(bk * Z[static_cast<size_t>(k - 1) * k + (k - 1)]);
  double eb = safety * std::max(std::fabs(th[k - 1]) + r_hi, std::fabs(th[0]) + r_lo);
  eb = std::min(eb, sum_abs);
  if (e_bound) *e_bound = eb;
  if (tmin) *tmin = th[0];
  if (tmax) *tmax = th[k - 1];
  return DACP_OK;
}

// Table entry of the on-chip spectral kernel for h (its flip tables built).
BatchSpec spectral_spec(dacp_ham h, int kind, int steps, const double *start, int64_t ld, double *out) {
  BatchSpec c;
  std::memset(&c, 0, sizeof(c));
  c.xc = h->onchip.xc;
  c.flips = h->onchip.flips;
  c.nflip = h->onchip.nflip;
  c.nplain = h->onchip.nplain;
  c.single = h->onchip.single;
  c.d64 = h->d64;
  c.L = h->L;
  c.kind = kind;
  c.steps = steps;
  c.start = start;
  c.ld = ld;
  c.out = out;
  return c;
}

dacp_status run_bound(dacp_ctx ctx, dacp_ham h, int steps, const double *v0, uint64_t seed, double safety,
                      double *e_bound, double *tmin, double *tmax) {
  const int64_t D = h->D;
  if (steps < 1) return set_err(ctx, DACP_E_INVALID, "bound: steps >= 1");
  steps = static_cast<int>(std::min<int64_t>(steps, D));
  hipStream_t s = ctx->stream;
  const bool onchip = onchip_fits(ctx, h, 1, 1, steps, 8.0);  // two more launches a step
  DevBuf bv, bp, bw, bs, dspec;
  const double *start = v0;
  if (!v0 || !onchip) {
    DACP_HIP(ctx, bv.alloc(D * sizeof(double)));
    if (v0) DACP_HIP(ctx, hipMemcpyAsync(bv.p, v0, D * sizeof(double), hipMemcpyDeviceToDevice, s));
    else DACP_HIP(ctx, dacp::launch_philox_gauss(bv.as<double>(), D, 1, seed, s));
    start = bv.as<double>();
  }
  std::vector<double> al, be;
  int taken = steps;
  double nv = 0.0;
  if (onchip) {
    DACP_TRY(onchip_order(ctx, h));
    DACP_HIP(ctx, bs.alloc((2 * steps + 2) * sizeof(double)));
    DACP_HIP(ctx, dspec.alloc(sizeof(BatchSpec)));
    const BatchSpec c = spectral_spec(h, 0, steps, start, 1, bs.as<double>());
    DACP_TRY(to_device(ctx, dspec.p, &c, sizeof(c)));
    DACP_HIP(ctx, dacp::launch_batch_spectral(dspec.as<BatchSpec>(), 1, h->L, s));
    std::vector<double> out(2 * steps + 2);
    DACP_TRY(to_host(ctx, out.data(), bs.p, out.size() * sizeof(double)));
    nv = out[2 * steps + 1];
    taken = static_cast<int>(out[2 * steps]);
    al.assign(out.begin(), out.begin() + steps);
    be.assign(out.begin() + steps, out.begin() + 2 * steps);
  } else {
    const int nb = dacp::scalar_blocks(D);
    DACP_HIP(ctx, bp.alloc(D * sizeof(double)));
    DACP_HIP(ctx, bw.alloc(D * sizeof(double)));
    DACP_HIP(ctx, bs.alloc((2 * steps + 2 * nb) * sizeof(double)));
    double *u = bv.as<double>(), *up = bp.as<double>(), *y = bw.as<double>();
    double *alpha = bs.as<double>(), *norms = alpha + steps, *pb = norms + steps, *pa = pb + nb;
    DACP_HIP(ctx, dacp::launch_sumsq(u, D, pb, s));
    for (int j = 0; j < steps; ++j) {
      DACP_TRY(step<double>(ctx, h, 1, u, 1, y, 1, 1.0));
      DACP_HIP(ctx, dacp::launch_lanczos_step(y, u, up, D, j, norms, alpha, pa, pb, s));
      std::swap(u, up);
    }
    std::vector<double> out(2 * steps + nb);
    DACP_TRY(to_host(ctx, out.data(), bs.p, out.size() * sizeof(double)));
    double last = 0.0;
    for (int q = 0; q < nb; ++q) last += out[2 * steps + q];
    al.assign(out.begin(), out.begin() + steps);
    be.assign(out.begin() + steps + 1, out.begin() + 2 * steps);  // beta_(j+1) couples v_j and v_(j+1)
    be.push_back(std::sqrt(std::max(last, 0.0)));
    nv = out[steps] * out[steps];
  }
  if (!(nv > 0.0)) return set_err(ctx, DACP_E_INVALID, "bound: zero start vector");
  // the recurrence ends at the first vanishing residual; what the device computed past it is unused
  int k = 0;
  while (k < taken) {
    if (!std::isfinite(al[k]) || !std::isfinite(be[k])) return set_err(ctx, DACP_E_NUMERIC, "bound: non-finite Lanczos");
    ++k;
    if (be[k - 1] <= 1e-300) break;
  }
  al.resize(k);
  be.resize(k);
  return lanczos_bound(ctx, al, be, safety, h->sum_abs, e_bound, tmin, tmax);
}

// ----------------------------------------------------------- KPM moments
// d[2 k] = <T_k R, T_k R> and d[2 k + 1] = <T_k R, T_(k-1) R> summed over the nvec columns, k = 0 .. M / 2.
dacp_status moment_dots(dacp_ctx ctx, dacp_ham h, double e_bound, int M, int nvec, const double *r,
                        std::vector<double> &d) {
  const int64_t D = h->D;
  hipStream_t s = ctx->stream;
  const int kmax = M / 2;
  d.assign(2 * kmax + 2, 0.0);
  if (onchip_fits(ctx, h, nvec, nvec, 0.5 * M, 4.0)) {  // a launch of dot products an order
    DACP_TRY(onchip_order(ctx, h));
    DevBuf dout, dspec;
    DACP_HIP(ctx, dout.alloc(static_cast<size_t>(M) * nvec * sizeof(double)));
    DACP_HIP(ctx, dspec.alloc(sizeof(BatchSpec) * nvec));
    std::vector<BatchSpec> specs;
    for (int q = 0; q < nvec; ++q) {
      specs.push_back(spectral_spec(h, 1, M, r + q, nvec, dout.as<double>() + static_cast<size_t>(M) * q));
      specs.back().inv_e = 1.0 / e_bound;
    }
    DACP_TRY(to_device(ctx, dspec.p, specs.data(), sizeof(BatchSpec) * nvec));
    DACP_HIP(ctx, dacp::launch_batch_spectral(dspec.as<BatchSpec>(), nvec, h->L, s));
    std::vector<double> out(static_cast<size_t>(M) * nvec);
    DACP_TRY(to_host(ctx, out.data(), dout.p, out.size() * sizeof(double)));
    for (int q = 0; q < nvec; ++q)  // entry i: <T_k, T_k> at i = 2 k, <T_(k+1), T_k> at i = 2 k + 1
      for (int i = 0; i < M; ++i) d[(i & 1) ? i + 2 : i] += out[static_cast<size_t>(q) * M + i];
    return DACP_OK;
  }
  ColGroups cg = column_groups(ctx, h, nvec, recurrence_group(ctx, h, nvec), 3, {8});
  DevBuf ba, bb, bp, part, sums;
  auto blocks = [&]() -> hipError_t {
    for (DevBuf *b : {&ba, &bb, &bp}) {
      const hipError_t e = (b != &bp || cg.fused) ? b->alloc(cg.elems(D) * sizeof(double)) : hipSuccess;
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  };
  hipError_t got_blocks = blocks();
  if (got_blocks == hipErrorOutOfMemory && cg.fused) {  // single applies do with two blocks, of one group's columns
    for (DevBuf *b : {&ba, &bb, &bp}) b->release();
    cg.fused = false;
    cg.g = std::min(cg.g, nvec);
    cg.per = 1;
    cg.tail = 0;
    got_blocks = blocks();
  }
  DACP_HIP(ctx, got_blocks);
  DACP_HIP(ctx, part.alloc(2 * static_cast<size_t>(kmax + 1) * 256 * sizeof(double)));
  DACP_HIP(ctx, sums.alloc(2 * static_cast<size_t>(kmax + 1) * sizeof(double)));
  std::vector<double> got(2 * kmax + 2);
  int64_t launches = 0;
  for (int g0 = 0; g0 < nvec; g0 += cg.cols(g0)) {
    const int nc = cg.cols(g0), gw = cg.width(g0), groups = cg.groups(g0);
    const int64_t n = D * gw * groups;  // zero columns add nothing
    const int nb = dacp::scalar_blocks(n);
    DACP_HIP(ctx, dacp::launch_split_cols(r + g0, nvec, nc, ba.as<double>(), D, gw, groups, s));
    auto visit = [&](int64_t k, const double *tk, const double *tk1) -> dacp_status {
      DACP_HIP(ctx, dacp::launch_dot_pair(tk, tk1, n, part.as<double>() + 2 * nb * k, s));
      return DACP_OK;
    };
    DACP_TRY(evolve_group(
        ctx, h, 1.0 / e_bound, kmax, gw, groups, nc, ba.as<double>(), bb.as<double>(), bp.as<double>(),
        [](int64_t) -> double * { return nullptr; }, 0, [](int64_t) { return true; }, visit,
        [](int64_t, int64_t) { return true; }, launches));
    DACP_HIP(ctx, dacp::launch_sum_pairs(part.as<double>(), kmax + 1, n, sums.as<double>(), s));
    DACP_TRY(to_host(ctx, got.data(), sums.p, got.size() * sizeof(double)));
    for (size_t i = 0; i < got.size(); ++i) d[i] += got[i];
  }
  return DACP_OK;
}

dacp_status run_moments(dacp_ctx ctx, dacp_ham h, double e_bound, int M, int nvec, const double *R, uint64_t seed,
                        double *mu) {
  const int64_t D = h->D;
  if (M < 1 || nvec < 1 || !(e_bound > 0.0)) return set_err(ctx, DACP_E_INVALID, "moments: bad arguments");
  DevBuf br;
  const double *r = R;
  if (!r) {
    DACP_HIP(ctx, br.alloc(static_cast<size_t>(D) * nvec * sizeof(double)));
    DACP_HIP(ctx, dacp::launch_philox_gauss(br.as<double>(), D, nvec, seed, ctx->stream));
    r = br.as<double>();
  }
  std::vector<double> d;
  DACP_TRY(moment_dots(ctx, h, e_bound, M, nvec, r, d));
  // mu_{2k} = 2 <T_k r, T_k r> - mu_0,  mu_{2k+1} = 2 <T_{k+1} r, T_k r> - mu_1
  const double n0 = d[0];
  mu[0] = 1.0;
  if (M > 1) mu[1] = d[3] / n0;
  for (int k = 1; 2 * k < M; ++k) {
    mu[2 * k] = 2.0 * d[2 * k] / n0 - mu[0];
    if (2 * k + 1 < M) mu[2 * k + 1] = 2.0 * d[2 * k + 3] / n0 - mu[1];
  }
  return DACP_OK;
}

}  // namespace

// =====================================================================  ABI

extern "C" {

const char *dacp_version(void) { return "dacp-mi355x 0.1 (gfx950)"; }

dacp_status dacp_create(int device, void *hip_stream, dacp_ctx *out) {
  if (!out) return DACP_E_INVALID;
  *out = nullptr;
  int ndev = 0;
  if (hipGetDeviceCount(&ndev) != hipSuccess || device < 0 || device >= ndev) return DACP_E_INVALID;
  if (hipSetDevice(device) != hipSuccess) return DACP_E_HIP;
  dacp_ctx c = new (std::nothrow) dacp_ctx_s();
  if (!c) return DACP_E_NOMEM;
  c->device = device;
  c->stream = static_cast<hipStream_t>(hip_stream);
  int cus = 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) == hipSuccess && cus > 0)
    c->num_cus = cus;
  // the device's copy of the allocation-free workspace, resolved once per device with it current;
  // a failure is reported by the entry point that needs it
  (void)dacp::noalloc_scratch_init(device);
  *out = c;
  return DACP_OK;
}

void dacp_destroy(dacp_ctx ctx) {
  if (!ctx) return;
  (void)hipSetDevice(ctx->device);
  if (ctx->red) (void)hipFree(ctx->red);
  if (ctx->red_out) (void)hipFree(ctx->red_out);
  delete ctx;
}

const char *dacp_last_error(dacp_ctx ctx) { return ctx ? ctx->err.c_str() : "null context"; }

dacp_status dacp_set_tile(dacp_ctx ctx, int tile_elems) {
  if (!ctx || tile_elems < 256 || tile_elems > 8192 || (tile_elems & (tile_elems - 1)))
    return set_err(ctx, DACP_E_INVALID, "tile_elems must be a power of two in [256, 8192]");
  ctx->tile_elems = tile_elems;
  return DACP_OK;
}

dacp_status dacp_tune(dacp_ctx ctx, const char *key, int value) {
  if (!ctx || !key) return DACP_E_INVALID;
  const std::string k(key);
  const bool pow2 = value > 0 && (value & (value - 1)) == 0;
  if (k == "tile") return dacp_set_tile(ctx, value);
  if (k == "pass_tile") {
    if (!pow2 || value < 512 || value > 16384) return set_err(ctx, DACP_E_INVALID, "pass_tile: power of two in [512, 16384]");
    ctx->pass_tile_elems = value;
    return DACP_OK;
  }
  if (k == "two_pass_L") {
    if (value < 0 || value > 31) return set_err(ctx, DACP_E_INVALID, "two_pass_L: 0..31");
    ctx->two_pass_min_L = value;
    return DACP_OK;
  }
  if (k == "fused") {
    if (value != 0 && value != 1) return set_err(ctx, DACP_E_INVALID, "fused: 0 or 1");
    ctx->fused_rec = value;
    return DACP_OK;
  }
  if (k == "dc") {
    if (value < 0) return set_err(ctx, DACP_E_INVALID, "dc: smallest size for divide and conquer (0 = never)");
    ctx->dc_min_n = value;
    return DACP_OK;
  }
  if (k == "filter_group_f64" || k == "filter_group_f32") {
    if (!pow2 || value > 64) return set_err(ctx, DACP_E_INVALID, k + ": power of two <= 64");
    (k == "filter_group_f64" ? ctx->filter_group_f64 : ctx->filter_group_f32) = value;
    return DACP_OK;
  }
  if (k == "rec_hi_w") {
    if (value != 0 && !(pow2 && value <= 8)) return set_err(ctx, DACP_E_INVALID, "rec_hi_w: 0 (automatic), 1, 2, 4 or 8");
    ctx->rec_hi_w = value;
    return DACP_OK;
  }
  if (k == "rec_threads") {
    if (value != 512 && value != 1024) return set_err(ctx, DACP_E_INVALID, "rec_threads: 512 or 1024");
    ctx->rec_threads = value;
    return DACP_OK;
  }
  if (k == "batch_workers") {
    if (value < 1 || value > 64) return set_err(ctx, DACP_E_INVALID, "batch_workers: 1..64");
    ctx->batch_workers = value;
    return DACP_OK;
  }
  if (k == "batch_eig") {
    if (value < 0 || value > 2) return set_err(ctx, DACP_E_INVALID, "batch_eig: 0, 1 or 2");
    ctx->batch_eig = value;
    return DACP_OK;
  }
  if (k == "moment_explicit") {
    if (value < 0 || value > 2) return set_err(ctx, DACP_E_INVALID, "moment_explicit: 0, 1 or 2");
    ctx->moment_explicit = value;
    return DACP_OK;
  }
  if (k == "beig_pipe") {
    if (value != 0 && value != 1) return set_err(ctx, DACP_E_INVALID, "beig_pipe: 0 or 1");
    ctx->beig_pipe = value;
    return DACP_OK;
  }
  if (k == "beig_sweeps") {
    if (value < 1 || value > 8) return set_err(ctx, DACP_E_INVALID, "beig_sweeps: 1..8");
    ctx->beig_sweeps = value;
    return DACP_OK;
  }
  if (k == "blocked") {
    if (value < 0) return set_err(ctx, DACP_E_INVALID, "blocked: size >= 0 (0 = never)");
    ctx->blocked_min_n = value;
    return DACP_OK;
  }
  if (k == "tri_spins") {
    if (value < 0 || value > (1 << 26)) return set_err(ctx, DACP_E_INVALID, "tri_spins: 0..2^26");
    ctx->tri_spins = value;
    return DACP_OK;
  }
  if (k == "project_whole") {
    if (value != 0 && value != 1) return set_err(ctx, DACP_E_INVALID, "project_whole: 0 or 1");
    ctx->project_whole = value;
    return DACP_OK;
  }
  if (k == "project_splitk") {
    if (value != 0 && value != 1) return set_err(ctx, DACP_E_INVALID, "project_splitk: 0 or 1");
    ctx->project_splitk = value;
    return DACP_OK;
  }
  if (k == "rec_xcd") {
    if (value < 0 || value > 3) return set_err(ctx, DACP_E_INVALID, "rec_xcd: 0..3 (bit 0 low pass, bit 1 high pass)");
    ctx->rec_xcd = value;
    return DACP_OK;
  }
  if (k == "rec_persist") {
    if (value < 0 || value > 8) return set_err(ctx, DACP_E_INVALID, "rec_persist: 0..8 workgroups per CU");
    ctx->rec_persist = value;
    return DACP_OK;
  }
  if (k == "rec_graph") {
    if (value < 0 || value > 256 || (value & 1)) return set_err(ctx, DACP_E_INVALID, "rec_graph: even, 0..256");
    ctx->rec_graph = value;
    return DACP_OK;
  }
  if (k == "rec_tile") {
    if (!pow2 || value < 1024 || value > 8192) return set_err(ctx, DACP_E_INVALID, "rec_tile: power of two in [1024, 8192]");
    ctx->rec_tile_elems = value;
    return DACP_OK;
  }
  if (k == "group") {
    if (!pow2 || value > 64) return set_err(ctx, DACP_E_INVALID, "group: power of two <= 64");
    ctx->group_default = value;
    return DACP_OK;
  }
  return set_err(ctx, DACP_E_INVALID, "unknown tuning key " + k);
}

dacp_status dacp_tune_get(dacp_ctx ctx, const char *key, int *value) {
  if (!ctx || !key || !value) return DACP_E_INVALID;
  const std::string k(key);
  if (k == "tile") *value = ctx->tile_elems;
  else if (k == "pass_tile") *value = ctx->pass_tile_elems;
  else if (k == "two_pass_L") *value = ctx->two_pass_min_L;
  else if (k == "fused") *value = ctx->fused_rec;
  else if (k == "dc") *value = ctx->dc_min_n;
  else if (k == "tri_spins") *value = ctx->tri_spins;
  else if (k == "group") *value = ctx->group_default;
  else if (k == "filter_group_f64") *value = ctx->filter_group_f64;
  else if (k == "filter_group_f32") *value = ctx->filter_group_f32;
  else if (k == "rec_hi_w") *value = ctx->rec_hi_w;
  else if (k == "rec_threads") *value = ctx->rec_threads;
  else if (k == "rec_tile") *value = ctx->rec_tile_elems;
  else if (k == "rec_persist") *value = ctx->rec_persist;
  else if (k == "rec_graph") *value = ctx->rec_graph;
  else if (k == "rec_xcd") *value = ctx->rec_xcd;
  else if (k == "project_whole") *value = ctx->project_whole;
  else if (k == "project_splitk") *value = ctx->project_splitk;
  else if (k == "blocked") *value = ctx->blocked_min_n;
  else if (k == "batch_eig") *value = ctx->batch_eig;
  else if (k == "moment_explicit") *value = ctx->moment_explicit;
  else if (k == "beig_pipe") *value = ctx->beig_pipe;
  else if (k == "beig_sweeps") *value = ctx->beig_sweeps;
  else if (k == "batch_workers") *value = ctx->batch_workers;
  else return set_err(ctx, DACP_E_INVALID, "unknown tuning key " + k);
  return DACP_OK;
}

dacp_status dacp_set_stream(dacp_ctx ctx, void *hip_stream) {
  if (!ctx) return DACP_E_INVALID;
  ctx->stream = static_cast<hipStream_t>(hip_stream);
  return DACP_OK;
}

dacp_status dacp_build_hamiltonian(dacp_ctx ctx, int L, int n_terms, const dacp_term *terms, dacp_ham *out) {
  if (!ctx || !out) return DACP_E_INVALID;
  *out = nullptr;
  if (L < 1 || L > 30) return set_err(ctx, DACP_E_INVALID, "L must be in [1, 30]");
  if (n_terms < 0 || (n_terms > 0 && !terms)) return set_err(ctx, DACP_E_INVALID, "bad term list");
  std::map<uint32_t, double> diag;                              // z-mask -> coefficient
  std::map<std::pair<uint32_t, uint32_t>, double> flips;        // (x-mask, z-mask) -> coefficient
  for (int t = 0; t < n_terms; ++t) {
    const dacp_term &tm = terms[t];
    if (tm.reserved != 0) return set_err(ctx, DACP_E_INVALID, "term " + std::to_string(t) + ": reserved != 0");
    if (!std::isfinite(tm.coeff)) return set_err(ctx, DACP_E_INVALID, "term " + std::to_string(t) + ": coefficient");
    if (tm.op_a > 3 || tm.op_b > 3) return set_err(ctx, DACP_E_INVALID, "term " + std::to_string(t) + ": op code");
    uint32_t x = 0, z = 0;
    int ny = 0;
    const int ops[2] = {tm.op_a, tm.op_b};
    const int sites[2] = {tm.site_a, tm.site_b};
    if (tm.op_b != DACP_I && tm.op_a != DACP_I && tm.site_a == tm.site_b)
      return set_err(ctx, DACP_E_INVALID, "term " + std::to_string(t) + ": two-body term on one site");
    for (int q = 0; q < 2; ++q) {
      if (ops[q] == DACP_I) continue;
      if (sites[q] >= L) return set_err(ctx, DACP_E_INVALID, "term " + std::to_string(t) + ": site >= L");
      const uint32_t bit = 1u << sites[q];
      if (ops[q] == DACP_X || ops[q] == DACP_Y) x |= bit;
      if (ops[q] == DACP_Z || ops[q] == DACP_Y) z |= bit;
      if (ops[q] == DACP_Y) ++ny;
    }
    if (ny % 2) return set_err(ctx, DACP_E_INVALID, "term " + std::to_string(t) + ": odd number of Y (imaginary)");
    // sigma^y = i sigma^x sigma^z, so a string with ny (even) Y factors carries i^ny = (-1)^(ny/2)
    const double c = ((ny / 2) % 2 ? -1.0 : 1.0) * tm.coeff;
    if (x == 0) diag[z] += c;
    else flips[{x, z}] += c;
  }
  dacp_ham h = new (std::nothrow) dacp_ham_s();
  if (!h) return set_err(ctx, DACP_E_NOMEM, "host allocation");
  h->ctx = ctx;
  h->L = L;
  h->D = int64_t(1) << L;
  std::vector<uint32_t> dz;
  std::vector<double> dc;
  for (auto &kv : diag) {
    if (kv.second == 0.0) continue;
    const double c2 = kv.second * kv.second;
    h->sum_abs += std::fabs(kv.second);
    h->sum_sq += c2;
    h->w_diag += c2;
    if (__builtin_popcount(kv.first) == 2) h->w_zz += c2;
    h->max_abs = std::max(h->max_abs, std::fabs(kv.second));
    ++h->n_strings;
    dz.push_back(kv.first);
    dc.push_back(kv.second);
  }
  for (auto &kv : flips) {
    if (kv.second == 0.0) continue;
    const double c2 = kv.second * kv.second;
    h->flips_host.push_back(FlipEntry{kv.first.first, kv.first.second, kv.second});
    h->sum_abs += std::fabs(kv.second);
    h->sum_sq += c2;
    if (__builtin_popcount(kv.first.first) == 1) h->w_flip1 += c2;
    h->max_abs = std::max(h->max_abs, std::fabs(kv.second));
    ++h->n_strings;
  }
  // a Pauli string commutes with prod_i sigma^x_i when it has an even number of Z and Y factors
  h->flip_sym = true;
  for (uint32_t zm : dz)
    if (__builtin_popcount(zm) % 2) h->flip_sym = false;
  for (const FlipEntry &f : h->flips_host)
    if (__builtin_popcount(f.zmask) % 2) h->flip_sym = false;
  std::stable_sort(h->flips_host.begin(), h->flips_host.end(),
                   [](const FlipEntry &a, const FlipEntry &b) { return a.xmask < b.xmask; });
  if (h->flips_host.size() > static_cast<size_t>(dacp::kMaxFlips)) {
    delete h;
    return set_err(ctx, DACP_E_INVALID, "too many distinct off-diagonal Pauli strings");
  }
  for (size_t i = 0; i < h->flips_host.size(); ++i) {
    const FlipEntry &f = h->flips_host[i];
    ++h->flip_counts.flips;
    h->flip_counts.masks += i == 0 || f.xmask != h->flips_host[i - 1].xmask;
    if (!onchip_single(f)) ++(f.zmask == 0 ? h->flip_counts.table_plain : h->flip_counts.table_signed);
  }
  auto fail = [&](hipError_t e, const char *what) {
    dacp_free_hamiltonian(h);
    return hip_err(ctx, e, what);
  };
  hipError_t e;
  if ((e = hipMalloc(&h->d64, h->D * sizeof(double))) != hipSuccess) return fail(e, "diag alloc");
  if ((e = hipMalloc(&h->d32, h->D * sizeof(float))) != hipSuccess) return fail(e, "diag alloc");
  const size_t nf = std::max<size_t>(1, h->flips_host.size());
  if ((e = hipMalloc(&h->flips, nf * sizeof(FlipEntry))) != hipSuccess) return fail(e, "flip alloc");
  if (!h->flips_host.empty() &&
      (e = hipMemcpy(h->flips, h->flips_host.data(), h->flips_host.size() * sizeof(FlipEntry),
                     hipMemcpyHostToDevice)) != hipSuccess)
    return fail(e, "flip upload");
  DevBuf bz, bc;
  const size_t nd = std::max<size_t>(1, dz.size());
  if ((e = bz.alloc(nd * sizeof(uint32_t))) != hipSuccess) return fail(e, "diag terms");
  if ((e = bc.alloc(nd * sizeof(double))) != hipSuccess) return fail(e, "diag terms");
  if (!dz.empty()) {
    if ((e = hipMemcpy(bz.p, dz.data(), dz.size() * sizeof(uint32_t), hipMemcpyHostToDevice)) != hipSuccess)
      return fail(e, "diag upload");
    if ((e = hipMemcpy(bc.p, dc.data(), dc.size() * sizeof(double), hipMemcpyHostToDevice)) != hipSuccess)
      return fail(e, "diag upload");
  }
  if ((e = dacp::launch_diag(bz.as<uint32_t>(), bc.as<double>(), static_cast<int>(dz.size()), h->D, h->d64, h->d32,
                             ctx->stream)) != hipSuccess)
    return fail(e, "diag kernel");
  if ((e = hipStreamSynchronize(ctx->stream)) != hipSuccess) return fail(e, "diag kernel");
  *out = h;
  return DACP_OK;
}

void dacp_free_hamiltonian(dacp_ham h) {
  if (!h) return;
  for (auto &so : h->split) {
    if (so.lo) (void)hipFree(so.lo);
    if (so.hi) (void)hipFree(so.hi);
  }
  for (auto &to : h->by_log2r)
    if (to.dev) (void)hipFree(to.dev);
  if (h->onchip.xc) (void)hipFree(h->onchip.xc);
  if (h->d64) (void)hipFree(h->d64);
  if (h->d32) (void)hipFree(h->d32);
  if (h->flips) (void)hipFree(h->flips);
  delete h;
}

dacp_status dacp_ham_info(dacp_ham h, int *L, double *sum_abs, double *sum_sq, int *n_flip_groups) {
  if (!h) return DACP_E_INVALID;
  if (L) *L = h->L;
  if (sum_abs) *sum_abs = h->sum_abs;
  if (sum_sq) *sum_sq = h->sum_sq;
  if (n_flip_groups) *n_flip_groups = static_cast<int>(h->flips_host.size());
  return DACP_OK;
}

dacp_status dacp_ham_flip_symmetry(dacp_ham h, int *flip_sym) {
  if (!h || !flip_sym) return DACP_E_INVALID;
  *flip_sym = h->flip_sym ? 1 : 0;
  return DACP_OK;
}

dacp_status dacp_apply(dacp_ctx ctx, dacp_ham h, int dtype, int b, const void *x, int64_t ldx, void *y, int64_t ldy) {
  if (!ctx || !h || !x || !y || b < 1 || ldx < b || ldy < b) return set_err(ctx, DACP_E_INVALID, "apply: bad args");
  if (dtype == DACP_F64)
    return step<double>(ctx, h, b, static_cast<const double *>(x), ldx, static_cast<double *>(y), ldy, 1.0);
  if (dtype == DACP_F32)
    return step<float>(ctx, h, b, static_cast<const float *>(x), ldx, static_cast<float *>(y), ldy, 1.0f);
  return set_err(ctx, DACP_E_INVALID, "apply: dtype");
}

dacp_status dacp_random_block(dacp_ctx ctx, int64_t D, int b, uint64_t seed, double *out) {
  if (!ctx || D < 1 || b < 1 || !out) return set_err(ctx, DACP_E_INVALID, "random_block: bad args");
  DACP_HIP(ctx, dacp::launch_philox_gauss(out, D, b, seed, ctx->stream));
  return DACP_OK;
}

dacp_status dacp_spectral_bound(dacp_ctx ctx, dacp_ham h, int steps, const double *v0, uint64_t seed, double safety,
                                double *e_bound, double *theta_min, double *theta_max) {
  if (!ctx || !h) return DACP_E_INVALID;
  return run_bound(ctx, h, steps, v0, seed, safety > 0.0 ? safety : 1.01, e_bound, theta_min, theta_max);
}

dacp_status dacp_dos_moments(dacp_ctx ctx, dacp_ham h, double e_bound, int n_moments, int nvec, const double *R,
                             uint64_t seed, double *mu_out) {
  if (!ctx || !h || !mu_out) return DACP_E_INVALID;
  return run_moments(ctx, h, e_bound, n_moments, nvec, R, seed, mu_out);
}

dacp_status dacp_filter(dacp_ctx ctx, dacp_ham h, const dacp_filter_params *p, const double *start, double *psi_out) {
  if (!ctx || !h || !p) return DACP_E_INVALID;
  return run_filter(ctx, h, p, start, psi_out);
}

dacp_status dacp_basis(dacp_ctx ctx, dacp_ham h, const dacp_basis_params *p, const double *psi_e, double *V,
                       int64_t ldv, int *m_out) {
  if (!ctx || !h || !p) return DACP_E_INVALID;
  return run_basis(ctx, h, p, psi_e, V, ldv, m_out, nullptr);
}

dacp_status dacp_basis_moments(dacp_ctx ctx, dacp_ham h, const dacp_basis_params *p, const double *psi_e, double *S,
                               double *P, int64_t ld, int *m_out) {
  if (!ctx || !h || !p) return DACP_E_INVALID;
  return run_moment_basis(ctx, h, p, psi_e, S, P, ld, m_out, nullptr);
}

dacp_status dacp_basis_stored_moments(dacp_ctx ctx, dacp_ham h, const dacp_basis_params *p, const double *psi_e,
                                      double *V, int64_t ldv, double *S, double *P, int64_t ld, int *m_out) {
  if (!ctx || !h || !p) return DACP_E_INVALID;
  return run_stored_moment_basis(ctx, h, p, psi_e, V, ldv, S, P, ld, m_out, nullptr, nullptr);
}

dacp_status dacp_project(dacp_ctx ctx, dacp_ham h, int m, const double *V, int64_t ldv, double *S, double *P,
                         int64_t ld) {
  if (!ctx || !h) return DACP_E_INVALID;
  return run_project(ctx, h, m, V, ldv, S, P, ld);
}

dacp_status dacp_rayleigh_ritz(dacp_ctx ctx, int m, const double *S, const double *P, int64_t ld, double eps,
                               double *theta_out, double *B_out, int *r_out) {
  if (!ctx || m < 1 || !S || !P || ld < m || !theta_out) return set_err(ctx, DACP_E_INVALID, "rayleigh_ritz: args");
  std::vector<double> theta;
  DevBuf bc;
  int r = 0;
  dacp_status st = run_rr(ctx, m, S, P, ld, eps, theta, B_out ? &bc : nullptr, &r);
  if (st) return st;
  std::copy(theta.begin(), theta.end(), theta_out);
  if (B_out) {
    DACP_HIP(ctx, hipMemcpyAsync(B_out, bc.p, static_cast<size_t>(r) * m * sizeof(double), hipMemcpyDeviceToDevice,
                                 ctx->stream));
    DACP_HIP(ctx, hipStreamSynchronize(ctx->stream));
  }
  if (r_out) *r_out = r;
  return DACP_OK;
}

dacp_status dacp_syev(dacp_ctx ctx, int n, double *A, int64_t ld, double *w, double *Zrows) {
  if (!ctx || n < 0 || (n > 0 && (!A || !w || ld < n))) return set_err(ctx, DACP_E_INVALID, "syev: args");
  return dacp::gpu_syev(ctx, n, A, ld, w, Zrows);
}

dacp_status dacp_syev_batched(dacp_ctx ctx, int count, const int *n, double *const *A, double *const *w,
                              double *const *Z) {
  if (!ctx || count < 0 || (count > 0 && (!n || !A || !w || !Z))) return set_err(ctx, DACP_E_INVALID, "syev_batched: args");
  for (int i = 0; i < count; ++i)
    if (n[i] < 1 || n[i] > dacp::kBatchEigMaxN || !A[i] || !w[i])
      return set_err(ctx, DACP_E_INVALID, "syev_batched: need 1 <= n <= 2048 and A, w for every matrix");
  try {
    std::vector<dacp::SyevJob> jobs;
    for (int i = 0; i < count; ++i) jobs.push_back({n[i], A[i], n[i], w[i], Z[i]});
    const dacp_status st = dacp::syev_jobs(ctx, jobs);
    if (st == DACP_E_NUMERIC) return set_err(ctx, DACP_E_CONVERGENCE, "syev_batched: no convergence, " + ctx->err);
    return st;
  } catch (...) {
    return set_err(ctx, DACP_E_NOMEM, "syev_batched: host allocation failed");
  }
}

dacp_status dacp_syev_batched_noalloc(dacp_ctx ctx, int count, const int *n, double *const *A, double *const *w,
                                      double *const *Z) {
  if (!ctx || count < 0 || (count > 0 && (!n || !A || !w || !Z)))
    return set_err(ctx, DACP_E_INVALID, "syev_batched_noalloc: args");
  for (int i = 0; i < count; ++i)
    if (n[i] < 1 || n[i] > dacp::kBatchEigMaxN || !A[i] || !w[i])
      return set_err(ctx, DACP_E_INVALID, "syev_batched_noalloc: need 1 <= n <= 2048 and A, w for every matrix");
  return dacp::batch_syev_noalloc(ctx, count, n, A, w, Z);
}

dacp_status dacp_gemm(dacp_ctx ctx, int transA, int transB, int64_t M, int64_t N, int64_t K, double alpha,
                      const double *A, int64_t lda, const double *B, int64_t ldb, double beta, double *C, int64_t ldc) {
  if (!ctx || M < 0 || N < 0 || K < 0 || !C) return set_err(ctx, DACP_E_INVALID, "gemm: args");
  DACP_HIP(ctx, dacp::launch_dgemm(transA ? 1 : 0, transB ? 1 : 0, M, N, K, alpha, A, lda, B, ldb, beta, C, ldc, 0,
                                   ctx->stream));
  return DACP_OK;
}

namespace {
// vecs_out (device, may be null): row s of the D x N block at vecs_out + s * ldvec gets component
// s of the unit Ritz vector of each returned value, in the order of eigs_out.
// phi_all (device, may be null): the candidates' Ritz vectors already formed (moment mode), D x
// n_sel0 with row stride n_sel0, column c for the c-th value in the (|theta|, theta) order; V and bc
// are then not read.
dacp_status accept_stage(dacp_ctx ctx, dacp_ham h, int N, double a, double n_w, double tol, double norm_est,
                         const double *V, int m, int r, const std::vector<double> &theta, const DevBuf &bc,
                         dacp_report &rep, double *eigs_out, double *err_out, int &accepted,
                         double *vecs_out = nullptr, int64_t ldvec = 0, const double *phi_all = nullptr) {
  const int64_t D = h->D;
  hipStream_t s = ctx->stream;
  dacp_status st;
  double t0 = now_ms();
  const std::vector<int> order0 = central_order(theta);
  const int n_sel0 = std::min(r, N + std::max(64, N / 8));
  // per Ritz value (index into theta): residual norm of the unit Ritz vector, squared norm of the
  // computed vector V b_j, and its Rayleigh quotient (NaN where not a candidate)
  std::vector<double> rho(r, NAN), phin2(r, 1.0), rq(theta);
  {
    const int cw = std::min(n_sel0, 512);
    DevBuf bsel, phi, hphi, dth, dperm;
    if (!phi_all) DACP_HIP(ctx, bsel.alloc(static_cast<size_t>(cw) * m * sizeof(double)));
    DACP_HIP(ctx, phi.alloc(static_cast<size_t>(D) * cw * sizeof(double)));
    DACP_HIP(ctx, hphi.alloc(static_cast<size_t>(D) * cw * sizeof(double)));
    DACP_HIP(ctx, dth.alloc(sizeof(double) * cw));
    DACP_HIP(ctx, dperm.alloc(sizeof(int) * cw));
    const int nblk = dacp::coldots_blocks(D, 2 * cw);
    st = ensure_red(ctx, static_cast<size_t>(nblk) * 3 * cw, 3 * cw);
    if (st) return st;
    std::vector<double> out(3 * cw);
    for (int c0 = 0; c0 < n_sel0; c0 += cw) {
      const int w = std::min(cw, n_sel0 - c0);
      std::vector<int> pr(order0.begin() + c0, order0.begin() + c0 + w);
      std::vector<double> th(w);
      for (int i = 0; i < w; ++i) th[i] = theta[pr[i]];
      DACP_TRY(to_device(ctx, dth.p, th.data(), sizeof(double) * w));
      if (phi_all) {
        DACP_HIP(ctx, dacp::launch_copy_cols(phi_all + c0, n_sel0, phi.as<double>(), w, D, w, s));
      } else {
        DACP_TRY(to_device(ctx, dperm.p, pr.data(), sizeof(int) * w));
        DACP_HIP(ctx, dacp::launch_gather_rows(bc.as<double>(), m, bsel.as<double>(), m, dperm.as<int>(), nullptr, w,
                                               m, s));
        // Phi = V B_sel  (D x w)
        DACP_HIP(ctx, dacp::launch_dgemm(0, 1, D, w, m, 1.0, V, m, bsel.as<double>(), m, 0.0, phi.as<double>(), w, 0,
                                         s));
      }
      st = step<double>(ctx, h, w, phi.as<double>(), w, hphi.as<double>(), w, 1.0);
      if (st) return st;
      DACP_HIP(ctx, dacp::launch_resid(phi.as<double>(), hphi.as<double>(), w, dth.as<double>(), D, w, ctx->red,
                                       dacp::coldots_blocks(D, 2 * w), ctx->red_out, s));
      DACP_TRY(to_host(ctx, out.data(), ctx->red_out, sizeof(double) * 3 * w));
      for (int i = 0; i < w; ++i) {
        const int j = pr[i];
        // r = H x - theta x with x = V b_j.  The Rayleigh quotient of the computed x is
        // theta + x.r / x.x; the residual taken about it is no larger than ||r|| / ||x||.
        rho[j] = std::sqrt(out[3 * i] / out[3 * i + 1]);
        phin2[j] = out[3 * i + 1];
        rq[j] = theta[j] + out[3 * i + 2] / out[3 * i + 1];
      }
    }
  }
  // The Ritz values of the projected problem carry the rounding of App. C's ill-conditioned
  // overlap matrix; the Rayleigh quotients of the computed Ritz vectors do not, and the residual
  // bounds hold for them.  The candidates therefore take their Rayleigh quotients, and the rule
  // runs on the re-sorted values; the candidates are the leading positions of the new (|theta|,
  // theta) order up to the first value that is not one.
  std::vector<int> srt(r);
  std::iota(srt.begin(), srt.end(), 0);
  std::stable_sort(srt.begin(), srt.end(), [&](int x, int y) { return rq[x] < rq[y]; });
  std::vector<double> ths(r);
  for (int i = 0; i < r; ++i) ths[i] = rq[srt[i]];
  const std::vector<int> order = central_order(ths);
  int n_sel = 0;
  while (n_sel < r && !std::isnan(rho[srt[order[n_sel]]])) ++n_sel;
  std::vector<double> rnorm(n_sel);
  for (int q = 0; q < n_sel; ++q) rnorm[q] = rho[srt[order[q]]];
  // acceptance (the rule is described at accept_rule)
  const AcceptResult ar = accept_rule(ths, order, n_sel, rnorm, a, tol);
  const std::vector<char> &ok = ar.ok, &ghost = ar.ghost;
  const std::vector<double> &est = ar.est;
  const std::vector<int> &core_idx = ar.core_idx;
  const double max_est = ar.max_est;
  const int n_ghost = ar.n_ghost;
  const int core = static_cast<int>(core_idx.size());
  if (verbose()) {
    int shown = 0;
    for (int q = 0; q < n_sel && shown < 6; ++q) {
      if (ok[order[q]] || ghost[order[q]]) continue;
      const int j = order[q];
      const double gl = j > 0 ? ths[j] - ths[j - 1] : INFINITY;
      const double gr = j + 1 < r ? ths[j + 1] - ths[j] : INFINITY;
      vlog("rejected #%d (|theta| rank %d): theta=%.10g r=%.3g est=%.3g gaps=(%.3g, %.3g) tol=%.3g", shown, q,
           ths[j], rnorm[q], est[q], gl, gr, tol);
      ++shown;
    }
    int n_ok = 0;
    for (int q = 0; q < n_sel; ++q) n_ok += ok[order[q]] ? 1 : 0;
    vlog("accepted (any position) %d of %d candidates; ghosts %d; contiguous core %d", n_ok, n_sel, n_ghost, core);
  }
  rep.n_candidates = n_sel;
  rep.n_accepted = core;
  rep.max_err_est = max_est;
  rep.n_ghost = n_ghost;
  rep.t_accept_ms = now_ms() - t0;
  vlog("acceptance done: %.1f ms, %d accepted of %d candidates", rep.t_accept_ms, core, n_sel);
  accepted = core;
  if (core >= N) {
    std::vector<std::tuple<double, double, int>> sel;  // (value, estimate, Ritz index into theta and B)
    for (int i = 0; i < N; ++i) {
      const int q = core_idx[i];
      sel.push_back({ths[order[q]], est[q], srt[order[q]]});
    }
    std::sort(sel.begin(), sel.end());
    for (int i = 0; i < N; ++i) {
      eigs_out[i] = std::get<0>(sel[i]);
      if (err_out) err_out[i] = std::get<1>(sel[i]);
    }
    rep.n_clusters_at_b = dacp::rules::clusters_at_width(eigs_out, N, tol, rep.b);
    if (vecs_out) {
      // Phi = V B_sel again for the returned values only, each column of B_sel scaled by
      // 1 / ||V b_j|| (the Ritz vectors are orthonormal only up to the S cut-off's rounding).
      const int cw = std::min(N, 512);
      DevBuf bsel, dperm, dscale;
      if (!phi_all) DACP_HIP(ctx, bsel.alloc(static_cast<size_t>(cw) * m * sizeof(double)));
      DACP_HIP(ctx, dperm.alloc(sizeof(int) * cw));
      DACP_HIP(ctx, dscale.alloc(sizeof(double) * cw));
      std::vector<int> pos0(r, -1);  // Ritz index -> candidate column of phi_all
      for (int c = 0; c < n_sel0; ++c) pos0[order0[c]] = c;
      for (int c0 = 0; c0 < N; c0 += cw) {
        const int w = std::min(cw, N - c0);
        std::vector<int> pr(w);
        std::vector<double> sc(w);
        for (int i = 0; i < w; ++i) {
          const int j = std::get<2>(sel[c0 + i]);
          pr[i] = phi_all ? pos0[j] : j;
          sc[i] = 1.0 / std::sqrt(phin2[j]);
        }
        DACP_TRY(to_device(ctx, dperm.p, pr.data(), sizeof(int) * w));
        DACP_TRY(to_device(ctx, dscale.p, sc.data(), sizeof(double) * w));
        if (phi_all) {
          DACP_HIP(ctx, dacp::launch_gather_cols(phi_all, n_sel0, dperm.as<int>(), dscale.as<double>(), D, w,
                                                 vecs_out + c0, ldvec, s));
        } else {
          DACP_HIP(ctx, dacp::launch_gather_rows(bc.as<double>(), m, bsel.as<double>(), m, dperm.as<int>(),
                                                 dscale.as<double>(), w, m, s));
          DACP_HIP(ctx, dacp::launch_dgemm(0, 1, D, w, m, 1.0, V, m, bsel.as<double>(), m, 0.0, vecs_out + c0, ldvec,
                                           0, s));
        }
        DACP_HIP(ctx, hipStreamSynchronize(s));  // the host staging of the next chunk reuses dperm / dscale
      }
    }
  }
  return DACP_OK;
}

dacp_status finish_projected(dacp_ctx ctx, dacp_ham h, int N, const dacp_opts &o, double a, double n_w, double tol,
                             double norm_est, const double *V, int m, DevBuf &sb, DevBuf &pb, dacp_report &rep,
                             double *eigs_out, double *err_out, int &accepted, const EigFn *eig, double *vecs_out,
                             int64_t ldvec);

dacp_status finish_basis(dacp_ctx ctx, dacp_ham h, int N, const dacp_opts &o, double a, double n_w, double tol,
                         double norm_est, const double *V, int m, dacp_report &rep, double *eigs_out, double *err_out,
                         int &accepted, const EigFn *eig = nullptr, double *vecs_out = nullptr,
                         int64_t ldvec = 0) {
  // projection (Sec. II.C)
  double t0 = now_ms();
  dacp_status st;
  DevBuf sb, pb;
  DACP_HIP(ctx, sb.alloc(static_cast<size_t>(m) * m * sizeof(double)));
  DACP_HIP(ctx, pb.alloc(static_cast<size_t>(m) * m * sizeof(double)));
  st = run_project(ctx, h, m, V, m, sb.as<double>(), pb.as<double>(), m);
  if (st) return st;
  rep.t_project_ms = now_ms() - t0;
  vlog("projection done: %.1f ms", rep.t_project_ms);
  return finish_projected(ctx, h, N, o, a, n_w, tol, norm_est, V, m, sb, pb, rep, eigs_out, err_out, accepted, eig,
                          vecs_out, ldvec);
}

// The subspace solve of S and P (released once reduced) and the acceptance on the Ritz vectors V b_j
// of the stored basis.
dacp_status finish_projected(dacp_ctx ctx, dacp_ham h, int N, const dacp_opts &o, double a, double n_w, double tol,
                             double norm_est, const double *V, int m, DevBuf &sb, DevBuf &pb, dacp_report &rep,
                             double *eigs_out, double *err_out, int &accepted, const EigFn *eig, double *vecs_out,
                             int64_t ldvec) {
  // generalised eigenproblem (App. C)
  double t0 = now_ms();
  dacp_status st;
  std::vector<double> theta;
  DevBuf bc;
  int r = 0;
  st = run_rr(ctx, m, sb.as<double>(), pb.as<double>(), m, o.eps > 0.0 ? o.eps : 1e-12, theta, &bc, &r, eig);
  if (st) return st;
  sb.release();
  pb.release();
  rep.rank = r;
  rep.t_gep_ms = now_ms() - t0;
  vlog("subspace solve done: %.1f ms, rank %d", rep.t_gep_ms, r);

  return accept_stage(ctx, h, N, a, n_w, tol, norm_est, V, m, r, theta, bc, rep, eigs_out, err_out, accepted,
                      vecs_out, ldvec);
}

// One attempt in moment mode (App. C, Eq. shift), after the filter: moments during an evolution to
// 2 k_n and S, P from them; the subspace solve; the candidates' Ritz vectors from a second
// evolution to k_n (no basis stored); then the acceptance on those vectors.  The evolution times
// of both passes go to t_evol_ms (S and P come out of the first), t_project_ms stays 0.
dacp_status moment_attempt(dacp_ctx ctx, dacp_ham h, int N, const dacp_opts &o, const dacp_basis_params &bp,
                           double a, double n_w, double tol, double norm_est, DevBuf &psi, dacp_report &rep,
                           double *eigs_out, double *err_out, int &accepted, double *vecs_out, int64_t ldvec) {
  const int64_t D = h->D;
  const int m = bp.b * (2 * bp.n + 1);
  double t0 = now_ms();
  EvolStats es;
  std::vector<double> theta;
  DevBuf bc;
  int r = 0;
  {
    DevBuf sb, pb;
    DACP_HIP(ctx, sb.alloc(static_cast<size_t>(m) * m * sizeof(double)));
    DACP_HIP(ctx, pb.alloc(static_cast<size_t>(m) * m * sizeof(double)));
    int m_got = 0;
    DACP_TRY(run_moment_basis(ctx, h, &bp, psi.as<double>(), sb.as<double>(), pb.as<double>(), m, &m_got, &es));
    rep.t_evol_ms = now_ms() - t0;
    vlog("moment evolution done: %.1f ms (%lld steps)", rep.t_evol_ms, static_cast<long long>(es.steps));
    t0 = now_ms();
    DACP_TRY(run_rr(ctx, m, sb.as<double>(), pb.as<double>(), m, o.eps > 0.0 ? o.eps : 1e-12, theta, &bc, &r));
  }
  rep.rank = r;
  rep.t_gep_ms = now_ms() - t0;
  rep.t_project_ms = 0.0;
  vlog("subspace solve done: %.1f ms, rank %d", rep.t_gep_ms, r);
  // candidates (the same set accept_stage takes) and their Ritz vectors by a second evolution
  const std::vector<int> order0 = central_order(theta);
  const int n_sel0 = std::min(r, N + std::max(64, N / 8));
  size_t free_b = 0, total_b = 0;
  DACP_HIP(ctx, hipMemGetInfo(&free_b, &total_b));
  const double need = static_cast<double>(D) * n_sel0 * 8.0;
  if (need > 0.9 * static_cast<double>(free_b))
    return set_err(ctx, DACP_E_NOMEM, "moment mode: the candidates' Ritz vectors (D x " + std::to_string(n_sel0) +
                                          " FP64) do not fit in free device memory");
  t0 = now_ms();
  DevBuf bsel, phi, dperm;
  DACP_HIP(ctx, bsel.alloc(static_cast<size_t>(n_sel0) * m * sizeof(double)));
  DACP_HIP(ctx, dperm.alloc(sizeof(int) * std::max(1, n_sel0)));
  DACP_TRY(to_device(ctx, dperm.p, order0.data(), sizeof(int) * n_sel0));
  DACP_HIP(ctx, dacp::launch_gather_rows(bc.as<double>(), m, bsel.as<double>(), m, dperm.as<int>(), nullptr, n_sel0, m,
                                         ctx->stream));
  DACP_HIP(ctx, phi.alloc(static_cast<size_t>(D) * n_sel0 * sizeof(double)));
  DACP_TRY(moment_ritz_vectors(ctx, h, &bp, psi.as<double>(), bsel.as<double>(), n_sel0, phi.as<double>(), &es));
  bsel.release();
  psi.release();
  rep.t_evol_ms += now_ms() - t0;
  rep.evol_steps = es.steps;
  rep.evol_launches = es.launches;
  rep.evol_kernel_ms = es.kernel_ms;
  rep.evol_group = es.group;
  vlog("Ritz vectors by the second evolution: %.1f ms", now_ms() - t0);
  return accept_stage(ctx, h, N, a, n_w, tol, norm_est, nullptr, m, r, theta, bc, rep, eigs_out, err_out, accepted,
                      vecs_out, ldvec, phi.as<double>());
}

dacp_status central_eigs(dacp_ctx ctx, dacp_ham h, int N, const dacp_opts *opts_in, double *eigs_out,
                         double *err_out, double *vecs_out, int64_t ldvec, int *n_out, dacp_report *report) {
  if (!ctx || !h || !eigs_out) return DACP_E_INVALID;
  const int64_t D = h->D;
  if (N < 1 || N > D) return set_err(ctx, DACP_E_INVALID, "central_eigs: need 1 <= N <= 2^L");
  if (vecs_out && ldvec < N) return set_err(ctx, DACP_E_INVALID, "central_eigpairs: need ldvec >= N");
  dacp_opts o;
  if (opts_in) o = *opts_in;
  else dacp_default_opts(&o);
  if (o.moment_mode < 0 || o.moment_mode > 2) return set_err(ctx, DACP_E_INVALID, "central_eigs: moment_mode is 0, 1 or 2");
  dacp_report rep;
  std::memset(&rep, 0, sizeof(rep));
  const double t_start = now_ms();

  // bound (Sec. III upper-bound estimator)
  double t0 = now_ms();
  double e_b = o.e_bound, th_lo = 0.0, th_hi = 0.0;
  dacp_status st;
  if (!(e_b > 0.0)) {
    st = run_bound(ctx, h, o.lanczos_steps > 0 ? o.lanczos_steps : 80, nullptr, o.seed ^ 0x5bd1e995ULL, 1.01, &e_b,
                   &th_lo, &th_hi);
    if (st) return st;
  } else {
    th_lo = -e_b;
    th_hi = e_b;
  }
  const double norm_est = std::max(std::fabs(th_lo), std::fabs(th_hi));
  const double tol = o.tol_rel * norm_est;
  std::vector<double> mu;
  if (!(o.a > 0.0)) {
    const int M = o.kpm_moments > 1 ? o.kpm_moments : 256;
    mu.assign(M, 0.0);
    st = run_moments(ctx, h, e_b, M, o.kpm_vectors > 0 ? o.kpm_vectors : 8, nullptr, o.seed ^ 0x2545f491ULL,
                     mu.data());
    if (st) return st;
  }
  rep.t_bound_ms = now_ms() - t0;
  double window_ratio = o.window_ratio > 0.0 ? o.window_ratio : 2.2;
  int accepted = 0;
  for (int attempt = 0;; ++attempt) {
    // window and orders (Sec. II.A, II.B, III)
    const Plan pl = make_plan(o, D, N, e_b, mu, window_ratio, attempt);
    const double n_w = pl.n_w, a_r = pl.a_r, a = pl.a;
    const int K = pl.K, b = pl.b, n = pl.n, m = pl.m;
    rep.e_bound = e_b;
    rep.a = a;
    rep.a_r = a_r;
    rep.K = K;
    rep.b = b;
    rep.n = n;
    rep.m = m;
    rep.retries = attempt;
    vlog("params: E_b=%.6g a=%.6g a_r=%.4g K=%d b=%d n=%d m=%d (attempt %d)", e_b, a, a_r, K, b, n, m, attempt);

    // filter (Sec. II.A)
    t0 = now_ms();
    DevBuf psi;
    DACP_HIP(ctx, psi.alloc(static_cast<size_t>(D) * b * sizeof(double)));
    dacp_filter_params fp;
    fp.e_bound = e_b;
    fp.a = a;
    fp.K = K;
    fp.b = b;
    fp.precision = o.precision;
    fp.fp64_tail = static_cast<int>(std::ceil(o.fp64_tail_frac * K));
    fp.seed = o.seed + static_cast<uint64_t>(attempt) * 0x9E3779B97F4A7C15ULL;
    DevBuf start;
    if (o.sectors && h->flip_sym && b >= 2) {
      // start columns split between the two eigenspaces of the global spin flip, which H keeps
      DACP_HIP(ctx, start.alloc(static_cast<size_t>(D) * b * sizeof(double)));
      DACP_HIP(ctx, dacp::launch_philox_gauss(start.as<double>(), D, b, fp.seed, ctx->stream));
      DACP_HIP(ctx, dacp::launch_parity_split(start.as<double>(), D, b, (b + 1) / 2, ctx->stream));
    }
    st = run_filter(ctx, h, &fp, start.p ? start.as<double>() : nullptr, psi.as<double>());
    if (st) return st;
    start.release();
    rep.t_filter_ms = now_ms() - t0;
    vlog("filter done: %.1f ms", rep.t_filter_ms);

    dacp_basis_params bp;
    bp.e_bound = e_b;
    bp.a = a;
    bp.n = n;
    bp.b = b;
    bp.group = o.group;
    if (o.moment_mode == 1) {
      st = moment_attempt(ctx, h, N, o, bp, a, n_w, tol, norm_est, psi, rep, eigs_out, err_out, accepted, vecs_out,
                          ldvec);
      if (st) return st;
      if (accepted >= N) {
        if (n_out) *n_out = N;
        rep.t_total_ms = now_ms() - t_start;
        if (report) *report = rep;
        return DACP_OK;
      }
      if (attempt >= o.max_retries) break;
      window_ratio *= 1.5;
      continue;
    }

    // evolution basis (Sec. II.B, App. B/C)
    t0 = now_ms();
    DevBuf vbuf;
    DACP_HIP(ctx, vbuf.alloc(static_cast<size_t>(D) * m * sizeof(double)));
    EvolStats es;
    int m_got = 0;
    if (o.moment_mode == 2) {
      // the uniform-grid basis stored, S and P from the anchors' moments (no V^T V, V^T H V)
      DevBuf sb, pb;
      DACP_HIP(ctx, sb.alloc(static_cast<size_t>(m) * m * sizeof(double)));
      DACP_HIP(ctx, pb.alloc(static_cast<size_t>(m) * m * sizeof(double)));
      double gram_ms = 0.0;
      st = run_stored_moment_basis(ctx, h, &bp, psi.as<double>(), vbuf.as<double>(), m, sb.as<double>(),
                                   pb.as<double>(), m, &m_got, &es, &gram_ms);
      if (st) return st;
      psi.release();
      rep.t_evol_ms = now_ms() - t0 - gram_ms;
      rep.t_project_ms = gram_ms;
      rep.evol_steps = es.steps;
      rep.evol_launches = es.launches;
      rep.evol_kernel_ms = es.kernel_ms;
      rep.evol_group = es.group;
      vlog("evolution done: %.1f ms (%lld launches); moments and S, P: %.1f ms", rep.t_evol_ms,
           static_cast<long long>(es.launches), gram_ms);
      st = finish_projected(ctx, h, N, o, a, n_w, tol, norm_est, vbuf.as<double>(), m, sb, pb, rep, eigs_out, err_out,
                            accepted, nullptr, vecs_out, ldvec);
      if (st) return st;
      if (ctx->moment_explicit == 2 || (ctx->moment_explicit == 1 && accepted < N)) {
        // The moments' rounding is not that of a Gram matrix of the stored panels, so a direction
        // at S's cut-off can be kept that the explicit products would drop, and its Ritz value
        // may end the core early.  Before widening the window, project the same basis explicitly.
        vlog("moment projection: core %d of %d; explicit products of the same basis", accepted, N);
        const int acc_moments = accepted;
        const double t_proj = rep.t_project_ms, t_gep = rep.t_gep_ms, t_acc = rep.t_accept_ms;
        st = finish_basis(ctx, h, N, o, a, n_w, tol, norm_est, vbuf.as<double>(), m, rep, eigs_out, err_out, accepted,
                          nullptr, vecs_out, ldvec);
        if (st) return st;
        vlog("explicit products: core %d (moments: %d)", accepted, acc_moments);
        rep.t_project_ms += t_proj;
        rep.t_gep_ms += t_gep;
        rep.t_accept_ms += t_acc;
      }
    } else {
      st = run_basis(ctx, h, &bp, psi.as<double>(), vbuf.as<double>(), m, &m_got, &es);
      if (st) return st;
      psi.release();
      rep.t_evol_ms = now_ms() - t0;
      rep.evol_steps = es.steps;
      rep.evol_launches = es.launches;
      rep.evol_kernel_ms = es.kernel_ms;
      rep.evol_group = es.group;
      vlog("evolution done: %.1f ms (%lld launches)", rep.t_evol_ms, static_cast<long long>(es.launches));

      st = finish_basis(ctx, h, N, o, a, n_w, tol, norm_est, vbuf.as<double>(), m, rep, eigs_out, err_out, accepted,
                        nullptr, vecs_out, ldvec);
      if (st) return st;
    }
    if (accepted >= N) {
      if (n_out) *n_out = N;
      rep.t_total_ms = now_ms() - t_start;
      if (report) *report = rep;
      return DACP_OK;
    }
    if (attempt >= o.max_retries) break;
    window_ratio *= 1.5;
  }
  if (n_out) *n_out = accepted;
  rep.t_total_ms = now_ms() - t_start;
  if (report) *report = rep;
  return set_err(ctx, DACP_E_WINDOW,
                 "only " + std::to_string(accepted) + " eigenvalues accepted near 0; widen the window");
}

}  // namespace

dacp_status dacp_central_eigs(dacp_ctx ctx, dacp_ham h, int N, const dacp_opts *opts, double *eigs_out,
                              double *err_out, int *n_out, dacp_report *report) {
  return central_eigs(ctx, h, N, opts, eigs_out, err_out, nullptr, 0, n_out, report);
}

dacp_status dacp_central_eigpairs(dacp_ctx ctx, dacp_ham h, int N, const dacp_opts *opts, double *eigs_out,
                                  double *err_out, double *vecs_out, int64_t ldvec, int *n_out,
                                  dacp_report *report) {
  if (!vecs_out) return ctx ? set_err(ctx, DACP_E_INVALID, "central_eigpairs: null vecs_out") : DACP_E_INVALID;
  return central_eigs(ctx, h, N, opts, eigs_out, err_out, vecs_out, ldvec, n_out, report);
}


namespace {
// Lanczos bounds (e_bs, norm_est) and Chebyshev moments (mus) of many realisations with every
// L <= 14: one launch of the batched spectral kernel per estimator (Sec. III estimators, the same
// start vectors as the single-realisation path).  o.e_bound > 0 skips the bounds, o.a > 0 the
// moments.
dacp_status batched_estimates(dacp_ctx ctx, int count, const dacp_ham *hams, const dacp_opts &o, int max_L,
                              std::vector<double> &e_bs, std::vector<double> &norm_est,
                              std::vector<std::vector<double>> &mus) {
  e_bs.assign(count, 0.0);
  norm_est.assign(count, 0.0);
  mus.assign(count, std::vector<double>());
  const int steps0 = o.lanczos_steps > 0 ? o.lanczos_steps : 80;
  const int M = o.kpm_moments > 1 ? o.kpm_moments : 256;
  const int nvec = o.kpm_vectors > 0 ? o.kpm_vectors : 8;
  std::vector<DevBuf> v0(count), out(count), R(count), mout(count);
  std::vector<BatchSpec> specs;
  std::vector<int> steps(count);
  const double tl0 = now_ms();
  if (!(o.e_bound > 0.0)) {
    for (int r = 0; r < count; ++r) {
      dacp_ham h = hams[r];
      const int64_t D = h->D;
      steps[r] = static_cast<int>(std::min<int64_t>(steps0, D));
      DACP_TRY(onchip_order(ctx, h));
      DACP_HIP(ctx, v0[r].alloc(D * sizeof(double)));
      DACP_HIP(ctx, dacp::launch_philox_gauss(v0[r].as<double>(), D, 1, o.seed ^ 0x5bd1e995ULL, ctx->stream));
      DACP_HIP(ctx, out[r].alloc((2 * steps[r] + 2) * sizeof(double)));
      specs.push_back(spectral_spec(h, 0, steps[r], v0[r].as<double>(), 1, out[r].as<double>()));
    }
    DevBuf dspecs;
    DACP_HIP(ctx, dspecs.alloc(sizeof(BatchSpec) * specs.size()));
    DACP_TRY(to_device(ctx, dspecs.p, specs.data(), sizeof(BatchSpec) * specs.size()));
    DACP_HIP(ctx, dacp::launch_batch_spectral(dspecs.as<BatchSpec>(), static_cast<int>(specs.size()), max_L,
                                              ctx->stream));
    const double tl = now_ms();
    std::vector<std::vector<double>> outs(count);
    for (int r = 0; r < count; ++r) {
      outs[r].resize(2 * steps[r] + 1);
      DACP_TRY(to_host(ctx, outs[r].data(), out[r].p, outs[r].size() * sizeof(double)));
    }
    // the bounds of the realisations on host threads (c = nullptr: no message), then the first
    // failure again on the context for its message
    auto bound_one = [&](dacp_ctx c, int r) -> dacp_status {
      const std::vector<double> &o2 = outs[r];
      const int k = static_cast<int>(o2[2 * steps[r]]);
      if (k < 1 || k > steps[r]) return set_err(c, DACP_E_NUMERIC, "batched: Lanczos run " + std::to_string(r));
      std::vector<double> al(o2.begin(), o2.begin() + k), be(o2.begin() + steps[r], o2.begin() + steps[r] + k);
      for (int j = 0; j < k; ++j)
        if (!std::isfinite(al[j]) || !std::isfinite(be[j]))
          return set_err(c, DACP_E_NUMERIC, "batched: non-finite Lanczos run " + std::to_string(r));
      double th_lo = 0.0, th_hi = 0.0;
      DACP_TRY(lanczos_bound(c, al, be, 1.01, hams[r]->sum_abs, &e_bs[r], &th_lo, &th_hi));
      norm_est[r] = std::max(std::fabs(th_lo), std::fabs(th_hi));
      return DACP_OK;
    };
    std::vector<dacp_status> bst(count, DACP_OK);
    dacp::host_parallel(count, ctx->batch_workers, [&](int r) { bst[r] = bound_one(nullptr, r); });
    for (int r = 0; r < count; ++r)
      if (bst[r]) return bound_one(ctx, r);
    vlog("batched Lanczos launch and bounds: %.1f ms (host part %.1f ms)", now_ms() - tl0, now_ms() - tl);
    specs.clear();
  } else {
    for (int r = 0; r < count; ++r) {
      e_bs[r] = o.e_bound;
      norm_est[r] = o.e_bound;
    }
  }
  if (!(o.a > 0.0)) {
    for (int r = 0; r < count; ++r) {
      dacp_ham h = hams[r];
      const int64_t D = h->D;
      DACP_TRY(onchip_order(ctx, h));
      DACP_HIP(ctx, R[r].alloc(static_cast<size_t>(D) * nvec * sizeof(double)));
      DACP_HIP(ctx, dacp::launch_philox_gauss(R[r].as<double>(), D, nvec, o.seed ^ 0x2545f491ULL, ctx->stream));
      DACP_HIP(ctx, mout[r].alloc(static_cast<size_t>(M) * nvec * sizeof(double)));
      for (int q = 0; q < nvec; ++q) {
        specs.push_back(spectral_spec(h, 1, M, R[r].as<double>() + q, nvec,
                                      mout[r].as<double>() + static_cast<int64_t>(M) * q));
        specs.back().inv_e = 1.0 / e_bs[r];
      }
    }
    DevBuf dspecs;
    DACP_HIP(ctx, dspecs.alloc(sizeof(BatchSpec) * specs.size()));
    DACP_TRY(to_device(ctx, dspecs.p, specs.data(), sizeof(BatchSpec) * specs.size()));
    DACP_HIP(ctx, dacp::launch_batch_spectral(dspecs.as<BatchSpec>(), static_cast<int>(specs.size()), max_L,
                                              ctx->stream));
    for (int r = 0; r < count; ++r) {
      std::vector<double> mo(static_cast<size_t>(M) * nvec);
      DACP_TRY(to_host(ctx, mo.data(), mout[r].p, mo.size() * sizeof(double)));
      auto tot = [&](int idx) {
        double t = 0.0;
        for (int q = 0; q < nvec; ++q) t += mo[static_cast<size_t>(q) * M + idx];
        return t;
      };
      std::vector<double> &mu = mus[r];
      mu.assign(M, 0.0);
      const double n0 = tot(0);
      mu[0] = 1.0;
      if (M > 1) mu[1] = tot(1) / n0;
      for (int k = 1; 2 * k < M; ++k) {
        mu[2 * k] = 2.0 * tot(2 * k) / n0 - mu[0];
        if (2 * k + 1 < M) mu[2 * k + 1] = 2.0 * tot(2 * k + 1) / n0 - mu[1];
      }
      for (double x : mu)
        if (!std::isfinite(x)) return set_err(ctx, DACP_E_NUMERIC, "batched: non-finite moments " + std::to_string(r));
    }
  }
  return DACP_OK;
}
}  // namespace

// The dense eigen-decompositions of the threads that finish batched realisations, solved together:
// each thread hands in all of its pending problems (possibly none) and waits; once every running
// thread has arrived the last one solves the whole round (syev_jobs: every stage one launch or a few
// for all of its matrices) and a new round starts.  Problems above that solver's size limit go
// through the per-problem one.
class EigRendezvous {
 public:
  struct Req {
    int n;
    double *A, *w, *Z;
  };
  explicit EigRendezvous(int workers, int device) : active_(workers), device_(device) {
    if (hipStreamCreateWithFlags(&stream_, hipStreamNonBlocking) != hipSuccess) stream_ = nullptr;
  }
  ~EigRendezvous() {
    if (stream_) (void)hipStreamDestroy(stream_);
  }
  // The matrices of reqs are complete at the current end of ctx's stream: the round's launches, on
  // the rendezvous' own stream, wait for that point through an event.  Results are complete on return.
  dacp_status solve_many(dacp_ctx ctx, const std::vector<Req> &reqs) {
    dacp_status big = DACP_OK;
    Arrival me;
    me.ctx = ctx;
    for (const Req &r : reqs) {
      if (dacp::syev_on_chip(ctx, r.n)) me.jobs.push_back({r.n, r.A, r.n, r.w, r.Z});
      else if (big == DACP_OK) big = dacp::gpu_syev(ctx, r.n, r.A, r.n, r.w, r.Z);
    }
    hipEvent_t ev = nullptr;
    hipError_t e = stream_ ? hipSuccess : hipErrorInvalidResourceHandle;
    if (e == hipSuccess) e = hipEventCreateWithFlags(&ev, hipEventDisableTiming);
    if (e == hipSuccess) e = hipEventRecord(ev, ctx->stream);
    if (e == hipSuccess) me.ready = ev;
    {
      std::unique_lock<std::mutex> lk(mu_);
      if (e != hipSuccess) me.jobs.clear();  // still arrive, so that the others are not held up
      arrived_.push_back(&me);
      const long gen = generation_;
      if (static_cast<int>(arrived_.size()) == active_) run_locked(ctx);
      else cv_.wait(lk, [&] { return generation_ != gen; });
    }
    if (ev) (void)hipEventDestroy(ev);  // the launch's wait on it is enqueued
    if (e != hipSuccess) return hip_err(ctx, e, "batched eigensolver: stream or event");
    return me.st != DACP_OK ? me.st : big;
  }
  // this thread has no further problems
  void leave(dacp_ctx ctx) {
    std::unique_lock<std::mutex> lk(mu_);
    --active_;
    if (active_ > 0 && static_cast<int>(arrived_.size()) == active_) run_locked(ctx);
  }

 private:
  struct Arrival {
    dacp_ctx ctx = nullptr;
    std::vector<dacp::SyevJob> jobs;
    hipEvent_t ready = nullptr;
    dacp_status st = DACP_OK;
  };
  // Runs the round (the lock held) and always ends it, so that no waiting thread is left behind.
  void run_locked(dacp_ctx ctx) {
    dacp_status st = DACP_OK;
    try {
      st = launch_round(ctx);
    } catch (...) {
      st = set_err(ctx, DACP_E_NOMEM, "batched eigensolver: host allocation failed");
    }
    // a round that failed half way may still be writing the waiting threads' buffers, which they release
    // to their own streams on return
    if (st != DACP_OK) (void)hipStreamSynchronize(stream_);
    for (Arrival *a : arrived_) {
      a->st = st;
      if (st != DACP_OK && a->ctx != ctx) a->ctx->err = ctx->err;
    }
    arrived_.clear();
    ++generation_;
    cv_.notify_all();
  }
  dacp_status launch_round(dacp_ctx ctx) {
    std::vector<dacp::SyevJob> jobs;
    for (Arrival *a : arrived_) jobs.insert(jobs.end(), a->jobs.begin(), a->jobs.end());
    if (jobs.empty()) return DACP_OK;
    // the launches go on the rendezvous' own stream, after every arrival's event; the leader's
    // context lends its error slot, its buffers come from the cache ordered on that stream
    dacp::AllocStream scope(stream_, device_);
    struct OwnStream {
      dacp_ctx c;
      hipStream_t own;
      ~OwnStream() { c->stream = own; }
    } restore{ctx, ctx->stream};
    ctx->stream = stream_;
    for (const Arrival *a : arrived_)
      if (a->ready) DACP_HIP(ctx, hipStreamWaitEvent(stream_, a->ready, 0));
    return dacp::syev_jobs(ctx, jobs);
  }
  std::mutex mu_;
  std::condition_variable cv_;
  std::vector<Arrival *> arrived_;
  int active_;
  int device_;
  hipStream_t stream_ = nullptr;
  long generation_ = 0;
};

namespace {
// Per-realisation bounds and windows given by the caller (the learned window): e_b[r] and a[r]
// replace the Lanczos bound and the density estimate; tolerances are taken relative to
// e_b[r] / (1 + margin).  A realisation whose bound proves too low (the evolution's norm guard) or
// whose core falls short is redone alone with the Lanczos / KPM estimates (model_fallback = 1).
struct BatchWindows {
  const double *e_b;
  const double *a;
  double margin;
};

dacp_status central_eigs_batched(dacp_ctx ctx, int count, const dacp_ham *hams, int N, const dacp_opts *opts_in,
                                 double *eigs_out, double *err_out, int *n_out, dacp_report *reports,
                                 const BatchWindows *given) {
  if (!ctx || count < 1 || !hams || !eigs_out || !n_out)
    return set_err(ctx, DACP_E_INVALID, "batched: need ctx, count >= 1, hams, eigs_out, n_out");
  int max_L = 0;
  for (int r = 0; r < count; ++r) {
    if (!hams[r]) return set_err(ctx, DACP_E_INVALID, "batched: null Hamiltonian " + std::to_string(r));
    if (hams[r]->L > 14)
      return set_err(ctx, DACP_E_INVALID, "batched: realisation " + std::to_string(r) + " has L > 14 (one column of "
                                          "2^L FP64 values must fit the 160 KB LDS of a compute unit)");
    if (N < 1 || N > hams[r]->D) return set_err(ctx, DACP_E_INVALID, "batched: need 1 <= N <= 2^L for every realisation");
    max_L = std::max(max_L, hams[r]->L);
  }
  // the context's device for this thread during the call (the worker threads select it too)
  struct DeviceScope {
    int prev = -1;
    explicit DeviceScope(int d) {
      if (hipGetDevice(&prev) != hipSuccess) prev = -1;
      if (prev != d) (void)hipSetDevice(d);
    }
    ~DeviceScope() {
      if (prev >= 0) (void)hipSetDevice(prev);
    }
  } device_scope(ctx->device);
  // every device buffer of the call, here and in the worker threads, from the block cache
  dacp::AllocStream pooled(ctx->stream, ctx->device);
  dacp_opts o;
  if (opts_in) o = *opts_in;
  else dacp_default_opts(&o);
  if (o.moment_mode < 0 || o.moment_mode > 2) return set_err(ctx, DACP_E_INVALID, "batched: moment_mode is 0, 1 or 2");
  const double t_start = now_ms();
  const double window_ratio = o.window_ratio > 0.0 ? o.window_ratio : 2.2;
  std::vector<dacp_report> rep(count);
  std::vector<double> norm_est(count), tol(count), e_bs(count);
  std::vector<Plan> plans(count);
  // bounds and densities of every realisation: one launch of Lanczos runs, then one launch of
  // Chebyshev-moment vectors (Sec. III estimators), same start vectors as the single path
  std::vector<std::vector<double>> mus(count);
  {
    const double tb = now_ms();
    if (given) {
      for (int r = 0; r < count; ++r) {
        e_bs[r] = given->e_b[r];
        norm_est[r] = e_bs[r] / (1.0 + given->margin);
      }
    } else {
      DACP_TRY(batched_estimates(ctx, count, hams, o, max_L, e_bs, norm_est, mus));
    }
    const double t_spec = now_ms() - tb;
    vlog("batched bounds and densities of %d realisations: %.1f ms", count, t_spec);
    const double tp = now_ms();
    dacp::host_parallel(count, ctx->batch_workers, [&](int r) {
      dacp_opts orr = o;
      if (given) orr.a = given->a[r];
      plans[r] = make_plan(orr, hams[r]->D, N, e_bs[r], mus[r], window_ratio, 0);
    });
    for (int r = 0; r < count; ++r) {
      std::memset(&rep[r], 0, sizeof(dacp_report));
      tol[r] = o.tol_rel * norm_est[r];
      const Plan &pl = plans[r];
      rep[r].e_bound = e_bs[r];
      rep[r].a = pl.a;
      rep[r].a_r = pl.a_r;
      rep[r].K = pl.K;
      rep[r].b = pl.b;
      rep[r].n = pl.n;
      rep[r].m = pl.m;
      rep[r].evol_group = 1;
      rep[r].t_bound_ms = t_spec;
    }
    vlog("batched plans: %.1f ms", now_ms() - tp);
  }
  const double t_setup = now_ms();

  // start blocks, bases and the column table of the persistent launch
  std::vector<DevBuf> psi(count), vb(count), ksd(count), ab(count), kad(count);
  // moment projection (moment_mode 2): panel orders on the uniform grid and the anchor orders
  const bool anchored = o.moment_mode == 2;
  std::vector<std::vector<int64_t>> orders_of(count), anchors_of(count);
  DevBuf flags;
  DACP_HIP(ctx, flags.alloc(sizeof(int) * count));
  DACP_HIP(ctx, hipMemsetAsync(flags.p, dacp::kBatchNoFlag & 0xff, sizeof(int) * count, ctx->stream));
  std::vector<BatchCol> cols;
  std::vector<double> col_work;
  for (int r = 0; r < count; ++r) {
    dacp_ham h = hams[r];
    const Plan &pl = plans[r];
    const int64_t D = h->D;
    DACP_HIP(ctx, psi[r].alloc(static_cast<size_t>(D) * pl.b * sizeof(double)));
    DACP_HIP(ctx, dacp::launch_philox_gauss(psi[r].as<double>(), D, pl.b, o.seed + static_cast<uint64_t>(r) * 0x9E3779B97F4A7C15ULL,
                                            ctx->stream));
    if (o.sectors && h->flip_sym && pl.b >= 2)
      DACP_HIP(ctx, dacp::launch_parity_split(psi[r].as<double>(), D, pl.b, (pl.b + 1) / 2, ctx->stream));
    DACP_HIP(ctx, vb[r].alloc(static_cast<size_t>(D) * pl.m * sizeof(double)));
    if (static_cast<double>(D) * pl.m * 8.0 >= 4294967296.0)
      return set_err(ctx, DACP_E_INVALID, "batched: basis of realisation " + std::to_string(r) + " exceeds 4 GiB");
    DACP_TRY(onchip_order(ctx, h));
    std::vector<int64_t> ks64;
    if (anchored) {
      const MomentPlan mp = moment_plan(pl.a_r, pl.n);
      for (int j = 1; j <= pl.n; ++j) ks64.push_back(mp.orders[2 * j]);
      orders_of[r] = mp.orders;
      anchors_of[r] = anchor_orders(mp.orders.back());
      const std::vector<int> ka(anchors_of[r].begin(), anchors_of[r].end());
      DACP_HIP(ctx, kad[r].alloc(sizeof(int) * ka.size()));
      DACP_TRY(to_device(ctx, kad[r].p, ka.data(), sizeof(int) * ka.size()));
      DACP_HIP(ctx, ab[r].alloc(static_cast<size_t>(D) * 2 * ka.size() * pl.b * sizeof(double)));
    } else {
      ks64 = sample_orders(pl.a_r, pl.n);
    }
    std::vector<int> ks(ks64.begin(), ks64.end());
    DACP_HIP(ctx, ksd[r].alloc(sizeof(int) * ks.size()));
    DACP_TRY(to_device(ctx, ksd[r].p, ks.data(), sizeof(int) * ks.size()));
    const int tail = (o.precision == DACP_F32) ? std::max(0, std::min(pl.K, static_cast<int>(std::ceil(o.fp64_tail_frac * pl.K)))) : pl.K;
    for (int j = 0; j < pl.b; ++j) {
      BatchCol c = onchip_col(h, dacp::kBatchBoth, e_bs[r], pl.a);
      c.psi0 = psi[r].as<double>() + j;
      c.ld_psi = pl.b;
      c.V = vb[r].as<double>() + j;
      c.ldv = pl.m;
      c.ks = ksd[r].as<int>();
      c.n_samples = pl.n;
      if (anchored) {
        c.n_anchor = static_cast<int>(anchors_of[r].size());
        c.lda = 2 * c.n_anchor * pl.b;
        c.A = ab[r].as<double>() + j;
        c.ka = kad[r].as<int>();
      }
      c.bound_flag = flags.as<int>() + r;
      c.K = pl.K;
      c.n32 = pl.K - tail;
      c.b = pl.b;
      cols.push_back(c);
      col_work.push_back((2.0 * pl.K + ks.back()) * static_cast<double>(D));
    }
  }
  // longest columns first (applies times elements), so the short ones fill in behind them
  {
    std::vector<int> order(cols.size());
    std::iota(order.begin(), order.end(), 0);
    std::stable_sort(order.begin(), order.end(), [&](int x, int y) { return col_work[x] > col_work[y]; });
    std::vector<BatchCol> sorted;
    for (int i : order) sorted.push_back(cols[i]);
    cols.swap(sorted);
  }
  DevBuf dcols;
  DACP_HIP(ctx, dcols.alloc(sizeof(BatchCol) * cols.size()));
  DACP_TRY(to_device(ctx, dcols.p, cols.data(), sizeof(BatchCol) * cols.size()));
  vlog("batched start blocks, bases and column table: %.1f ms", now_ms() - t_setup);
  const double tb0 = now_ms();
  DACP_HIP(ctx, dacp::launch_batch_chebyshev(dcols.as<BatchCol>(), static_cast<int>(cols.size()), max_L, ctx->stream));
  std::vector<int> flag(count);
  DACP_TRY(to_host(ctx, flag.data(), flags.p, sizeof(int) * count));
  const double t_batch = now_ms() - tb0;
  vlog("batched filter + evolution: %d columns of %d realisations in %.1f ms", static_cast<int>(cols.size()), count,
       t_batch);
  std::vector<char> redo(count, 0);  // given windows only: realisations redone with Lanczos / KPM
  for (int r = 0; r < count; ++r) {
    psi[r].release();
    rep[r].t_evol_ms = t_batch;
    if (flag[r] != dacp::kBatchNoFlag && given) {
      redo[r] = 1;
      vb[r].release();
      continue;
    }
    if (flag[r] != dacp::kBatchNoFlag)
      return set_err(ctx, DACP_E_BOUNDS, "batched: realisation " + std::to_string(r) +
                                             ": |T_k(H/e_bound)| grew above 1; e_bound is below ||H||");
  }

  // projection, subspace solve and acceptance: realisations spread over worker contexts, each
  // with its own stream, so the small GEMMs and eigen-solves of different realisations overlap
  const int nw = std::max(1, std::min(count, ctx->batch_workers));
  std::vector<dacp_ctx_s> wctx(nw);
  std::vector<dacp_status> wst(count, DACP_OK);
  std::vector<std::string> werr(count);
  std::vector<int> acc(count, 0);
  for (int w = 0; w < nw; ++w) {
    dacp_ctx_s &c = wctx[w];
    c.worker_of(*ctx);
    DACP_HIP(ctx, hipStreamCreateWithFlags(&c.stream, hipStreamNonBlocking));
  }
  EigRendezvous rendezvous(nw, ctx->device);
  std::vector<char> has_left(nw, 0);  // the worker has left the rendezvous
  // The matrices of a round share every launch of the eigensolver, so that even a few of them (a retry
  // round) finish sooner together: one of n = 1000 takes 6 ms alone, 4 and 8 take 9.4 and 11.3 ms together.
  const bool batch_eig = ctx->batch_eig == 2 || (ctx->batch_eig == 1 && count > dacp::kBatchEigMinCount);
  // Each thread finishes its realisations r = w, w + nw, ...: with the batched eigensolver, stage by
  // stage (projection; eig(S) for all of them in the shared launch; U and H~; eig(H~) likewise;
  // Ritz vectors and acceptance), else one realisation after another.
  auto worker = [&](int w) {
    (void)hipSetDevice(ctx->device);
    dacp_ctx wc = &wctx[w];
    dacp::AllocStream pooled_w(wc->stream, ctx->device);
    const double eps = o.eps > 0.0 ? o.eps : 1e-12;
    if (!batch_eig) {
      for (int r = w; r < count; r += nw) {
        if (redo[r]) continue;
        const Plan &pl = plans[r];
        double *eo = eigs_out + static_cast<int64_t>(r) * N;
        double *ee = err_out ? err_out + static_cast<int64_t>(r) * N : nullptr;
        if (anchored) {
          const double t0 = now_ms();
          DevBuf sb, pb;
          hipError_t e = sb.alloc(static_cast<size_t>(pl.m) * pl.m * sizeof(double));
          if (e == hipSuccess) e = pb.alloc(static_cast<size_t>(pl.m) * pl.m * sizeof(double));
          wst[r] = e != hipSuccess ? hip_err(wc, e, "batched finish: allocation")
                                   : anchor_projection(wc, hams[r], orders_of[r], anchors_of[r], ab[r].as<double>(),
                                                       vb[r].as<double>(), pl.m, pl.b, e_bs[r], sb.as<double>(),
                                                       pb.as<double>(), pl.m, nullptr);
          ab[r].release();
          rep[r].t_project_ms = now_ms() - t0;
          if (wst[r] == DACP_OK)
            wst[r] = finish_projected(wc, hams[r], N, o, pl.a, pl.n_w, tol[r], norm_est[r], vb[r].as<double>(), pl.m,
                                      sb, pb, rep[r], eo, ee, acc[r], nullptr, nullptr, 0);
          // as in the single call: the explicit products of the same basis before any retry round
          if (wst[r] == DACP_OK && (ctx->moment_explicit == 2 || (ctx->moment_explicit == 1 && acc[r] < N)))
            wst[r] = finish_basis(wc, hams[r], N, o, pl.a, pl.n_w, tol[r], norm_est[r], vb[r].as<double>(), pl.m,
                                  rep[r], eo, ee, acc[r]);
        } else {
          wst[r] = finish_basis(wc, hams[r], N, o, pl.a, pl.n_w, tol[r], norm_est[r], vb[r].as<double>(), pl.m, rep[r],
                                eo, ee, acc[r]);
        }
        if (wst[r]) werr[r] = wc->err;
        vb[r].release();
      }
      rendezvous.leave(wc);
      has_left[w] = 1;
      return;
    }
    struct Fin {
      DevBuf sb, pb, awork, zs, uc, ht, yc, bc;
      std::vector<double> lam, theta;
      int rank = 0;
      double t0 = 0.0;
    };
    std::vector<int> mine;
    for (int r = w; r < count; r += nw)
      if (!redo[r]) mine.push_back(r);
    std::vector<Fin> F(mine.size());
    auto fail = [&](int r, dacp_status st) {
      wst[r] = st;
      werr[r] = wc->err;
    };
    auto alive = [&](int r) { return wst[r] == DACP_OK; };
    // projection (Sec. II.C), then a copy of S for the eigensolver
    for (size_t i = 0; i < mine.size(); ++i) {
      const int r = mine[i];
      const int m = plans[r].m;
      Fin &f = F[i];
      const double t0 = now_ms();
      hipError_t e = f.sb.alloc(static_cast<size_t>(m) * m * sizeof(double));
      if (e == hipSuccess) e = f.pb.alloc(static_cast<size_t>(m) * m * sizeof(double));
      if (e == hipSuccess) e = f.awork.alloc(static_cast<size_t>(m) * m * sizeof(double));
      if (e == hipSuccess) e = f.zs.alloc(static_cast<size_t>(m) * m * sizeof(double));
      if (e != hipSuccess) {
        fail(r, hip_err(wc, e, "batched finish: allocation"));
        continue;
      }
      dacp_status st =
          anchored ? anchor_projection(wc, hams[r], orders_of[r], anchors_of[r], ab[r].as<double>(), vb[r].as<double>(),
                                       m, plans[r].b, e_bs[r], f.sb.as<double>(), f.pb.as<double>(), m, nullptr)
                   : run_project(wc, hams[r], m, vb[r].as<double>(), m, f.sb.as<double>(), f.pb.as<double>(), m);
      ab[r].release();
      if (st == DACP_OK) {
        e = dacp::launch_copy_cols(f.sb.as<double>(), m, f.awork.as<double>(), m, m, m, wc->stream);
        if (e != hipSuccess) st = hip_err(wc, e, "batched finish: copy");
      }
      if (st) {
        fail(r, st);
        continue;
      }
      f.lam.assign(m, 0.0);
      rep[r].t_project_ms = now_ms() - t0;
      f.t0 = now_ms();
    }
    // eig(S) of every realisation in one launch
    {
      std::vector<EigRendezvous::Req> reqs;
      for (size_t i = 0; i < mine.size(); ++i)
        if (alive(mine[i]))
          reqs.push_back({plans[mine[i]].m, F[i].awork.as<double>(), F[i].lam.data(), F[i].zs.as<double>()});
      const dacp_status st = rendezvous.solve_many(wc, reqs);
      if (st)
        for (int r : mine)
          if (alive(r)) fail(r, st);
    }
    // U = V~ Lambda~^(-1/2), H~ = U^T P U
    for (size_t i = 0; i < mine.size(); ++i) {
      const int r = mine[i];
      if (!alive(r)) continue;
      Fin &f = F[i];
      const int m = plans[r].m;
      dacp_status st = rr_reduce(wc, m, f.lam, f.zs.as<double>(), f.pb.as<double>(), m, eps, f.uc, f.ht, &f.rank);
      if (st == DACP_OK) {
        const hipError_t e = f.yc.alloc(static_cast<size_t>(f.rank) * f.rank * sizeof(double));
        if (e != hipSuccess) st = hip_err(wc, e, "batched finish: allocation");
      }
      if (st) {
        fail(r, st);
        continue;
      }
      f.sb.release();
      f.pb.release();
      f.awork.release();
      f.zs.release();
      f.theta.assign(f.rank, 0.0);
    }
    // eig(H~) of every realisation in one launch
    {
      std::vector<EigRendezvous::Req> reqs;
      for (size_t i = 0; i < mine.size(); ++i)
        if (alive(mine[i])) reqs.push_back({F[i].rank, F[i].ht.as<double>(), F[i].theta.data(), F[i].yc.as<double>()});
      const dacp_status st = rendezvous.solve_many(wc, reqs);
      if (st)
        for (int r : mine)
          if (alive(r)) fail(r, st);
    }
    rendezvous.leave(wc);
    has_left[w] = 1;
    // B, Ritz vectors and acceptance
    for (size_t i = 0; i < mine.size(); ++i) {
      const int r = mine[i];
      Fin &f = F[i];
      if (alive(r)) {
        const Plan &pl = plans[r];
        dacp_status st = rr_back(wc, pl.m, f.rank, f.yc.as<double>(), f.uc.as<double>(), f.theta, &f.bc);
        if (st == DACP_OK) {
          rep[r].rank = f.rank;
          rep[r].t_gep_ms = now_ms() - f.t0;
          f.ht.release();
          f.yc.release();
          f.uc.release();
          st = accept_stage(wc, hams[r], N, pl.a, pl.n_w, tol[r], norm_est[r], vb[r].as<double>(), pl.m, f.rank,
                            f.theta, f.bc, rep[r], eigs_out + static_cast<int64_t>(r) * N,
                            err_out ? err_out + static_cast<int64_t>(r) * N : nullptr, acc[r]);
        }
        // as in the single call: with the moment projection, the explicit products of the same
        // basis (solved on this thread's stream) before any retry round
        if (st == DACP_OK && anchored &&
            (ctx->moment_explicit == 2 || (ctx->moment_explicit == 1 && acc[r] < N))) {
          for (DevBuf *b : {&f.sb, &f.pb, &f.awork, &f.zs, &f.uc, &f.ht, &f.yc, &f.bc}) b->release();
          st = finish_basis(wc, hams[r], N, o, pl.a, pl.n_w, tol[r], norm_est[r], vb[r].as<double>(), pl.m, rep[r],
                            eigs_out + static_cast<int64_t>(r) * N,
                            err_out ? err_out + static_cast<int64_t>(r) * N : nullptr, acc[r]);
        }
        if (st) fail(r, st);
      }
      for (DevBuf *b : {&f.sb, &f.pb, &f.awork, &f.zs, &f.uc, &f.ht, &f.yc, &f.bc}) b->release();
      vb[r].release();
    }
  };
  // A host exception in a worker (an allocation) fails its realisations; the thread still leaves
  // the rendezvous so that the others are not held up.
  auto guarded = [&](int w) {
    try {
      worker(w);
    } catch (...) {
      for (int r = w; r < count; r += nw) {
        wst[r] = DACP_E_NOMEM;
        werr[r] = "batched finish: host allocation failed";
      }
      if (!has_left[w]) rendezvous.leave(&wctx[w]);
    }
  };
  std::vector<std::thread> threads;
  for (int w = 1; w < nw; ++w) threads.emplace_back(guarded, w);
  guarded(0);
  for (auto &t : threads) t.join();
  for (int w = 0; w < nw; ++w) {
    if (wctx[w].red) (void)hipFree(wctx[w].red);
    if (wctx[w].red_out) (void)hipFree(wctx[w].red_out);
    (void)hipStreamDestroy(wctx[w].stream);
  }
  for (int r = 0; r < count; ++r)
    if (wst[r]) return set_err(ctx, wst[r], "batched: realisation " + std::to_string(r) + ": " + werr[r]);

  // Realisations whose core fell short are redone together in one more batched call with a 1.5x
  // wider window, a basis ratio 0.2 higher and new start blocks (up to opts.max_retries times);
  // with given windows, the short ones and those whose
  // bound proved too low are redone with the Lanczos / KPM estimates (the method's own estimators
  // are the fallback) and the same window ratio.
  dacp_status worst = DACP_OK;
  std::vector<int> again;
  for (int r = 0; r < count; ++r) {
    n_out[r] = acc[r] >= N ? N : acc[r];
    if (acc[r] >= N && !redo[r]) {
      if (given) rep[r].model_used = 1;
      continue;
    }
    again.push_back(r);
  }
  if (!again.empty() && (given || o.max_retries > 0)) {
    const int na = static_cast<int>(again.size());
    std::vector<dacp_ham> sub(na);
    for (int i = 0; i < na; ++i) sub[i] = hams[again[i]];
    dacp_opts o2 = o;
    if (!given) {
      // a wider window, a denser basis (a core usually ends at a pair of close levels left with
      // large residuals: more basis vectors per level resolve it) and new start blocks
      o2.window_ratio = window_ratio * 1.5;
      o2.basis_ratio = (o.basis_ratio > 0.0 ? o.basis_ratio : 1.5) + 0.2;
      o2.seed = o.seed + 0xD1B54A32D192ED03ULL;
      o2.max_retries = o.max_retries - 1;
    }
    std::vector<double> e2(static_cast<size_t>(na) * N), r2e(err_out ? static_cast<size_t>(na) * N : 0);
    std::vector<int> n2(na, 0);
    std::vector<dacp_report> rp2(na);
    vlog("batched: %d realisations redone (%s)", na, given ? "Lanczos / KPM fallback" : "wider window");
    worst = central_eigs_batched(ctx, na, sub.data(), N, &o2, e2.data(), err_out ? r2e.data() : nullptr, n2.data(),
                                 rp2.data(), nullptr);
    if (worst != DACP_OK && worst != DACP_E_WINDOW) return worst;
    for (int i = 0; i < na; ++i) {
      const int r = again[i];
      std::copy(e2.begin() + static_cast<int64_t>(i) * N, e2.begin() + static_cast<int64_t>(i + 1) * N,
                eigs_out + static_cast<int64_t>(r) * N);
      if (err_out)
        std::copy(r2e.begin() + static_cast<int64_t>(i) * N, r2e.begin() + static_cast<int64_t>(i + 1) * N,
                  err_out + static_cast<int64_t>(r) * N);
      rp2[i].retries += 1;
      rp2[i].t_bound_ms += rep[r].t_bound_ms;
      if (given) {
        rp2[i].model_used = 1;
        rp2[i].model_fallback = 1;
      }
      rep[r] = rp2[i];
      n_out[r] = n2[i];
    }
  } else if (!again.empty()) {
    worst = DACP_E_WINDOW;
  }
  const double total = now_ms() - t_start;
  for (int r = 0; r < count; ++r) {
    rep[r].t_total_ms = total;
    if (reports) reports[r] = rep[r];
  }
  if (worst != DACP_OK) return set_err(ctx, worst, "batched: some realisations fell short of N accepted eigenvalues");
  return DACP_OK;
}
}  // namespace

dacp_status dacp_central_eigs_batched(dacp_ctx ctx, int count, const dacp_ham *hams, int N, const dacp_opts *opts_in,
                                      double *eigs_out, double *err_out, int *n_out, dacp_report *reports) {
  return central_eigs_batched(ctx, count, hams, N, opts_in, eigs_out, err_out, n_out, reports, nullptr);
}

dacp_status dacp_autotune_batched(dacp_ctx ctx, int count, const dacp_ham *hams, int N, const dacp_opts *opts_in,
                                  int sample_every, dacp_opts *best, double *best_s) {
  if (!ctx || count < 1 || !hams || !best || sample_every < 1)
    return set_err(ctx, DACP_E_INVALID, "autotune_batched: need ctx, count >= 1, hams, best, sample_every >= 1");
  dacp_opts o;
  if (opts_in) o = *opts_in;
  else dacp_default_opts(&o);
  // a sample of the realisations, always including one of every L present (the largest L sets the
  // length of the shared launch)
  std::vector<dacp_ham> smp;
  std::set<int> Ls;
  for (int r = 0; r < count; ++r) {
    if (!hams[r]) return set_err(ctx, DACP_E_INVALID, "autotune_batched: null Hamiltonian");
    const bool first_of_L = Ls.insert(hams[r]->L).second;
    if (first_of_L || r % sample_every == 0) smp.push_back(hams[r]);
  }
  const int ns = static_cast<int>(smp.size());
  std::vector<double> e(static_cast<size_t>(ns) * N);
  std::vector<int> n_out(ns);
  std::vector<dacp_report> rp(ns);
  double best_t = INFINITY;
  bool found = false;
  for (double wr : {2.2, 2.5, 2.8})
    for (double br : {1.3, 1.5})
      for (double kf : {12.0, 18.0}) {
        dacp_opts c = o;
        c.window_ratio = wr;
        c.basis_ratio = br;
        c.kfac = kf;
        const double t0 = now_ms();
        const dacp_status st = central_eigs_batched(ctx, ns, smp.data(), N, &c, e.data(), nullptr, n_out.data(),
                                                    rp.data(), nullptr);
        const double t = now_ms() - t0;
        vlog("autotune_batched: window %.1f basis %.1f kfac %.0f: status %d, %.1f ms", wr, br, kf,
             static_cast<int>(st), t);
        if (st == DACP_E_WINDOW) continue;
        if (st != DACP_OK) return st;
        if (t < best_t) {
          best_t = t;
          *best = c;
          found = true;
        }
      }
  if (!found) return set_err(ctx, DACP_E_WINDOW, "autotune_batched: no candidate reached N");
  if (best_s) *best_s = best_t * 1e-3;
  return DACP_OK;
}

dacp_status dacp_window_features(dacp_ham h, double *f) {
  if (!h || !f) return DACP_E_INVALID;
  const double sig2 = h->sum_sq;
  if (!(sig2 > 0.0) || h->n_strings < 1) return DACP_E_INVALID;
  const double sig = std::sqrt(sig2);
  const double L = h->L;
  f[0] = L / 20.0;
  f[1] = std::log(sig);
  f[2] = h->w_diag / sig2;
  f[3] = h->w_zz / sig2;
  f[4] = h->w_flip1 / sig2;
  f[5] = h->max_abs / sig;
  f[6] = h->sum_abs / (sig * std::sqrt(static_cast<double>(h->n_strings)));
  f[7] = std::log(static_cast<double>(h->n_strings)) / std::log(L * (L + 1.0) / 2.0 + 2.0 * L);
  return DACP_OK;
}

dacp_status dacp_window_labels(dacp_ctx ctx, int count, const dacp_ham *hams, const dacp_opts *opts, double *labels) {
  if (!ctx || count < 1 || !hams || !labels) return DACP_E_INVALID;
  dacp_opts o;
  if (opts) o = *opts;
  else dacp_default_opts(&o);
  o.e_bound = 0.0;  // labels come from the estimators themselves
  o.a = 0.0;
  int max_L = 0;
  for (int r = 0; r < count; ++r) {
    if (!hams[r] || !(hams[r]->sum_sq > 0.0)) return set_err(ctx, DACP_E_INVALID, "window_labels: bad Hamiltonian");
    max_L = std::max(max_L, hams[r]->L);
  }
  std::vector<double> e_bs(count), norm_est(count);
  std::vector<std::vector<double>> mus(count);
  {
    // L <= 14 in one batched launch per estimator, the rest one by one
    std::vector<dacp_ham> small;
    std::vector<int> where;
    int ml = 0;
    for (int r = 0; r < count; ++r)
      if (hams[r]->L <= 14) {
        small.push_back(hams[r]);
        where.push_back(r);
        ml = std::max(ml, hams[r]->L);
      }
    if (!small.empty()) {
      std::vector<double> eb2, ne2;
      std::vector<std::vector<double>> mu2;
      DACP_TRY(batched_estimates(ctx, static_cast<int>(small.size()), small.data(), o, ml, eb2, ne2, mu2));
      for (size_t q = 0; q < small.size(); ++q) {
        e_bs[where[q]] = eb2[q];
        mus[where[q]] = mu2[q];
      }
    }
    const int M = o.kpm_moments > 1 ? o.kpm_moments : 256;
    for (int r = 0; r < count; ++r) {
      if (hams[r]->L <= 14) continue;
      double lo = 0.0, hi = 0.0;
      DACP_TRY(run_bound(ctx, hams[r], o.lanczos_steps > 0 ? o.lanczos_steps : 80, nullptr, o.seed ^ 0x5bd1e995ULL, 1.01,
                         &e_bs[r], &lo, &hi));
      mus[r].assign(M, 0.0);
      DACP_TRY(run_moments(ctx, hams[r], e_bs[r], M, o.kpm_vectors > 0 ? o.kpm_vectors : 8, nullptr,
                           o.seed ^ 0x2545f491ULL, mus[r].data()));
    }
  }
  const double a_r0 = 0.02;
  for (int r = 0; r < count; ++r) {
    const double sig = std::sqrt(hams[r]->sum_sq);
    const double D = static_cast<double>(hams[r]->D);
    const double rho0 = kpm_count(mus[r], hams[r]->D, a_r0) / (2.0 * a_r0 * e_bs[r]);
    if (!(rho0 > 0.0)) return set_err(ctx, DACP_E_NUMERIC, "window_labels: no levels near 0 in realisation " + std::to_string(r));
    labels[2 * r] = std::log(e_bs[r] / (sig * std::sqrt(2.0 * hams[r]->L * M_LN2)));
    labels[2 * r + 1] = std::log(rho0 * std::sqrt(2.0 * M_PI) * sig / D);
  }
  return DACP_OK;
}

dacp_status dacp_central_eigs_learned(dacp_ctx ctx, dacp_ham h, dacp_mlp model, double bound_margin, int N,
                                      const dacp_opts *opts_in, double *eigs_out, double *err_out, int *n_out,
                                      dacp_report *report) {
  if (!ctx || !h || !model || !eigs_out || !(bound_margin >= 0.0))
    return set_err(ctx, DACP_E_INVALID, "central_eigs_learned: need ctx, h, model, eigs_out, bound_margin >= 0");
  dacp_opts o;
  if (opts_in) o = *opts_in;
  else dacp_default_opts(&o);
  const double t0 = now_ms();
  double f[DACP_WINDOW_FEATURES], y[2];
  if (dacp_window_features(h, f) != DACP_OK) return set_err(ctx, DACP_E_INVALID, "central_eigs_learned: features");
  DACP_TRY(dacp_mlp_predict(ctx, model, 1, f, y));
  const double sig = std::sqrt(h->sum_sq);
  const double D = static_cast<double>(h->D);
  double e_b = std::min((1.0 + bound_margin) * sig * std::sqrt(2.0 * h->L * M_LN2) * std::exp(y[0]), h->sum_abs);
  const double rho0 = D * std::exp(y[1]) / (std::sqrt(2.0 * M_PI) * sig);
  const double n_w = std::min(D, std::ceil((o.window_ratio > 0.0 ? o.window_ratio : 2.2) * N));
  double a = std::min(0.95 * e_b, n_w / (2.0 * rho0));
  dacp_opts o2 = o;
  o2.e_bound = e_b;
  o2.a = a;
  o2.tol_rel = o.tol_rel / (1.0 + bound_margin);  // tolerance relative to the unwidened bound
  const double t_pred = now_ms() - t0;
  vlog("learned window: E_b=%.6g a=%.6g (prediction %.2f ms)", e_b, a, t_pred);
  dacp_report r1;
  std::memset(&r1, 0, sizeof(r1));
  int got = 0;
  dacp_status st = (std::isfinite(e_b) && std::isfinite(a) && a > 0.0 && e_b > a)
                       ? dacp_central_eigs(ctx, h, N, &o2, eigs_out, err_out, &got, &r1)
                       : DACP_E_WINDOW;
  r1.model_used = 1;
  r1.t_bound_ms = t_pred;
  if (st == DACP_E_BOUNDS || st == DACP_E_WINDOW || st == DACP_E_NUMERIC) {
    vlog("learned window failed (status %d): Lanczos / KPM fallback", static_cast<int>(st));
    dacp_report r2;
    std::memset(&r2, 0, sizeof(r2));
    st = dacp_central_eigs(ctx, h, N, &o, eigs_out, err_out, &got, &r2);
    r2.model_used = 1;
    r2.model_fallback = 1;
    r2.t_total_ms = now_ms() - t0;
    r1 = r2;
  } else {
    r1.t_total_ms = now_ms() - t0;
  }
  if (n_out) *n_out = got;
  if (report) *report = r1;
  return st;
}

dacp_status dacp_central_eigs_batched_learned(dacp_ctx ctx, int count, const dacp_ham *hams, dacp_mlp model,
                                              double bound_margin, int N, const dacp_opts *opts_in, double *eigs_out,
                                              double *err_out, int *n_out, dacp_report *reports) {
  if (!ctx || count < 1 || !hams || !model || !eigs_out || !n_out || !(bound_margin >= 0.0))
    return set_err(ctx, DACP_E_INVALID, "batched_learned: need ctx, count >= 1, hams, model, eigs_out, n_out, margin >= 0");
  dacp_opts o;
  if (opts_in) o = *opts_in;
  else dacp_default_opts(&o);
  const double t0 = now_ms();
  std::vector<double> f(static_cast<size_t>(count) * DACP_WINDOW_FEATURES), y(2 * static_cast<size_t>(count));
  for (int r = 0; r < count; ++r) {
    if (!hams[r] || dacp_window_features(hams[r], f.data() + static_cast<size_t>(r) * DACP_WINDOW_FEATURES) != DACP_OK)
      return set_err(ctx, DACP_E_INVALID, "batched_learned: features of realisation " + std::to_string(r));
  }
  DACP_TRY(dacp_mlp_predict(ctx, model, count, f.data(), y.data()));
  std::vector<double> e_b(count), a(count);
  for (int r = 0; r < count; ++r) {
    const dacp_ham h = hams[r];
    const double sig = std::sqrt(h->sum_sq);
    const double D = static_cast<double>(h->D);
    e_b[r] = std::min((1.0 + bound_margin) * sig * std::sqrt(2.0 * h->L * M_LN2) * std::exp(y[2 * r]), h->sum_abs);
    const double rho0 = D * std::exp(y[2 * r + 1]) / (std::sqrt(2.0 * M_PI) * sig);
    const double n_w = std::min(D, std::ceil((o.window_ratio > 0.0 ? o.window_ratio : 2.2) * N));
    a[r] = std::min(0.95 * e_b[r], n_w / (2.0 * rho0));
    if (!(std::isfinite(e_b[r]) && std::isfinite(a[r]) && a[r] > 0.0 && e_b[r] > a[r]))
      return set_err(ctx, DACP_E_NUMERIC, "batched_learned: prediction for realisation " + std::to_string(r));
  }
  const double t_pred = now_ms() - t0;
  vlog("batched learned windows of %d realisations: %.2f ms", count, t_pred);
  BatchWindows bw{e_b.data(), a.data(), bound_margin};
  dacp_opts o2 = o;
  o2.tol_rel = o.tol_rel;  // relative to e_b / (1 + margin), see BatchWindows
  const dacp_status st = central_eigs_batched(ctx, count, hams, N, &o2, eigs_out, err_out, n_out, reports, &bw);
  if (reports)
    for (int r = 0; r < count; ++r)
      if (!reports[r].model_fallback) reports[r].t_bound_ms = t_pred;
  return st;
}

dacp_status dacp_autotune(dacp_ctx ctx, dacp_ham h, int b, int steps, int *best_group, double *best_us_per_column_step) {
  if (!ctx || !h || b < 1 || steps < 4) return set_err(ctx, DACP_E_INVALID, "autotune: need b >= 1, steps >= 4");
  const int64_t D = h->D;
  struct Cand {
    int group, threads, tile, hi_w;
  };
  std::vector<Cand> cands;
  // smaller tiles only where the launch would otherwise leave compute units idle (below 2^19 rows)
  for (int g = 1; g <= std::min(b, 16); g *= 2)
    for (int th : {512, 1024})
      for (int tile : {1024, 2048, 4096, 8192}) {
        if (tile < 4096 && D >= (int64_t(1) << 19)) continue;
        for (int w : {0, 1, 2}) cands.push_back({g, th, tile, w});
      }
  const int saved_threads = ctx->rec_threads, saved_tile = ctx->rec_tile_elems, saved_w = ctx->rec_hi_w;
  // unit start columns; E_b = sum |c| >= ||H||; a_r = pi / steps puts the first sample pair at k = steps
  DevBuf psi, V;
  const int gmax = std::min(b, 16);
  const int bmax =
      static_cast<int>(std::max<int64_t>(gmax, std::min<int64_t>(b, dacp::rules::kRecCacheBytes / (D * 24))));
  DACP_HIP(ctx, psi.alloc(static_cast<size_t>(D) * bmax * sizeof(double)));
  DACP_HIP(ctx, V.alloc(static_cast<size_t>(D) * 3 * bmax * sizeof(double)));
  double best = INFINITY;
  Cand bc = cands.front();
  int n_ready = 0;
  std::set<int64_t> shapes;
  for (const Cand &c : cands) {
    ctx->rec_threads = c.threads;
    ctx->rec_tile_elems = c.tile;
    ctx->rec_hi_w = c.hi_w;
    // time each distinct launch shape once: knob settings that resolve to the same fused plan (or
    // to the unfused apply for this width) run the same kernels
    int ncol = c.group;
    {
      int lb = 0, wf = 0;
      const bool fz = fused_plan(ctx, h, c.group, lb, wf, 8);
      // the columns one launch advances (the general kernels': one group)
      const ColGroups cg = column_groups(ctx, h, bmax, c.group, 3, {8});
      ncol = cg.fused ? std::min(bmax, cg.g * cg.per) : c.group;
      const int64_t key = fz ? ((static_cast<int64_t>(c.group) * 4096 + c.threads) * 64 + lb) * 16 + wf : -c.group;
      if (!shapes.insert(key).second) continue;
    }
    dacp_basis_params bp;
    bp.e_bound = h->sum_abs;
    bp.a = h->sum_abs * M_PI / steps;
    bp.n = 1;
    bp.b = ncol;
    bp.group = c.group;
    if (!(bp.a < bp.e_bound)) continue;
    if (ncol != n_ready) {  // a [D][ncol] start block
      DACP_HIP(ctx, dacp::launch_philox_gauss(psi.as<double>(), D, ncol, 12345, ctx->stream));
      DACP_TRY(normalise_cols(ctx, psi.as<double>(), D, ncol));
      n_ready = ncol;
    }
    EvolStats es;
    int m = 0;
    // first call loads the kernels and the flip tables, the second is timed
    // (the kernels that the knobs are for, also where a call would take the on-chip one)
    dacp_status st = run_basis(ctx, h, &bp, psi.as<double>(), V.as<double>(), 3 * ncol, &m, &es, false);
    if (st == DACP_OK) st = run_basis(ctx, h, &bp, psi.as<double>(), V.as<double>(), 3 * ncol, &m, &es, false);
    if (st != DACP_OK || es.steps < 1) {
      ctx->err.clear();
      continue;
    }
    const double us = es.kernel_ms * 1e3 / (static_cast<double>(es.steps) * ncol);
    vlog("autotune: group %d threads %d tile %d hi_w %d: %.3f us per column-step", c.group, c.threads, c.tile, c.hi_w,
         us);
    if (us < best) {
      best = us;
      bc = c;
    }
  }
  // keep the winner
  if (!std::isfinite(best)) {
    ctx->rec_threads = saved_threads;
    ctx->rec_tile_elems = saved_tile;
    ctx->rec_hi_w = saved_w;
    return set_err(ctx, DACP_E_NUMERIC, "autotune: no candidate ran");
  }
  ctx->group_default = bc.group;
  ctx->rec_threads = bc.threads;
  ctx->rec_tile_elems = bc.tile;
  ctx->rec_hi_w = bc.hi_w;
  if (best_group) *best_group = bc.group;
  if (best_us_per_column_step) *best_us_per_column_step = best;
  return DACP_OK;
}

}  // extern "C"
