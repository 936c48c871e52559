// Host runtime of the C ABI declared in include/lssvm.h: argument checks,
// workspace carve-up, the CG driver loop (Sec. III-B) and the bias step
// (Eq. (15)). Every numeric step runs in the gfx950 kernels of kernels.hip;
// this file only validates, sequences launches and reads back scalars.
#include "lssvm.h"
#include "lssvm_error.h"
#include "lssvm_internal.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

namespace lssvm {

thread_local std::string g_last_error;

int fail(int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  std::vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_last_error = buf;
  return code;
}

void clear_error() { g_last_error.clear(); }

namespace {

#define LSSVM_HIP(call)                                                                  \
  do {                                                                                   \
    hipError_t e_ = (call);                                                              \
    if (e_ != hipSuccess)                                                                \
      return fail(LSSVM_EHIP, "%s failed: %s (%s:%d)", #call, hipGetErrorString(e_),     \
                  __FILE__, __LINE__);                                                   \
  } while (0)

#define LSSVM_TRY(expr)      \
  do {                       \
    int rc_ = (expr);        \
    if (rc_ != LSSVM_OK) return rc_; \
  } while (0)

constexpr size_t kAlign = 256;
// Supported sizes: the tile visit order takes n^2 / 8192 bytes (2 GiB at
// n = 2^22) and packs tile indices in 16 bits; a panel's buffer span stays
// below 4 GiB up to 2^21 features.
constexpr int64_t kMaxPoints = int64_t(1) << 22;
constexpr int64_t kMaxFeatures = int64_t(1) << 21;

// LSSVM_LOG=1 in the environment: one stderr line per batch of CG iterations
// and one per finished training (read once per process).
bool log_enabled() {
  static const bool on = [] {
    const char* v = std::getenv("LSSVM_LOG");
    return v && *v && std::strcmp(v, "0") != 0;
  }();
  return on;
}
constexpr int64_t kReplaceEvery = 50;  // residual recomputed every 50th iteration
// The products of linear trainings are so nearly exact that the CG recurrence
// goes on falling below the residual that fp64 iterates can have (4096 x 1024,
// eps 1e-13: 7.7e-14 at iteration 161 against a true 1.3e-12). So for an eps
// below this, a linear training of passes recomputes the residual as soon as the
// recurrence meets eps, and converges on that (or at the last iteration allowed). Left
// to the next 50th iteration a recurrence of few features falls as far as the
// underflow, where d^T Q~ d = 0 ends CG as a breakdown.
constexpr double kTrustedEps = 1e-12;

inline int64_t round_up(int64_t v, int64_t m) { return (v + m - 1) / m * m; }
inline size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

using clock_t_ = std::chrono::steady_clock;
inline double ms_since(clock_t_::time_point t0) {
  return std::chrono::duration<double, std::milli>(clock_t_::now() - t0).count();
}

// Padded sizes for n points of d features (element type T).
struct Geometry {
  int64_t n, d, N;  // N = n - 1 unknowns of the reduced system
  int64_t tile, bk;
  int64_t ld;       // points per feature row of the layout (>= n, multiple of tile)
  int64_t d_pad;    // features, an even number of staged blocks
  int64_t plan_nkb; // feature blocks of bk the tile plans count (even)
  int64_t nT;       // tiles per edge of the reduced system
  int64_t NP;       // nT * tile: padded length of every CG vector
  int64_t nb;       // blocks of the CG vector kernels over NP (block partials per reduction)
  // polynomial and RBF kernels:
  int64_t tail_q;      // tiles of the last partial round that tail_plan splits (or 0)
  int64_t tail_split;  // ... over this many workgroups each
  int64_t part_q;      // the tiles, the last of the visit order, that are split
  int64_t part_split;  // ... over this many workgroups each
  int64_t part_blocks; // ... of so many staged blocks (even; the last has what is left)
};

#ifndef LSSVM_FUSED_SMALL
#define LSSVM_FUSED_SMALL 1
#endif
// Small problems run each CG iteration (except the residual recomputations)
// as one launch: the product's tiles and, in the last workgroup, the vector
// work (launch_tiles_cg). Their iterations are launch-bound: four dependent
// launches of a few microseconds each against a product of ~10 us. Up to
// kFusedMaxNP, where both are measured.
inline bool fused_iteration(const Geometry& g, int32_t kernel) {
  const int64_t most = kernel == LSSVM_LINEAR ? kFusedMaxLinear : kFusedMaxNP;
  return LSSVM_FUSED_SMALL && g.NP <= most;
}

// Linear products run in two passes over the points, w = X^T p and X w (k_lin_w,
// k_lin_rows): O(n d) in place of the tiles' O(n^2 d). Measured per CG iteration,
// fp64: 4096 x 1024 258 us with tiles and 30 us so, 20011 x 301 1840 and 38,
// 600 x 3000 196 and 24. Only up to 1025 points of few features, where an
// iteration on tiles is one launch of a block or two per workgroup, do the four
// launches lose: 1000 x 100 22.4 us against 21.3, 1000 x 30 23.6 against 15.7;
// at 600 x 200 they win, 20 against 38, at 300 x 400 20 against 61.
inline bool linear_passes(const Geometry& g, int32_t kernel) {
  constexpr int64_t kFusedFeatures = 128;
  return kernel == LSSVM_LINEAR && !(fused_iteration(g, kernel) && g.d <= kFusedFeatures);
}

inline int64_t tri_count(int64_t nT) { return nT * (nT + 1) / 2; }

// Workgroups resident at once in a tile launch: two per CU on 256 CUs.
constexpr int64_t kCUs = 256;
constexpr int64_t kResidentTiles = 2 * kCUs;
#ifndef LSSVM_LINEAR_SPLIT_MAX
#define LSSVM_LINEAR_SPLIT_MAX 16
#endif

// The tiles beyond the last full round of resident workgroups run one per
// CU and take about as long as a whole round. When they are at most a
// quarter round, each is split over S (4..16) workgroups that park their
// partial inner products, and one more launch sums them per tile and
// finishes it: the tail then costs ~1/S of a round plus the fixup.
inline void tail_plan(int64_t nT, int64_t nkb, int64_t* q, int64_t* split) {
  const int64_t Q = tri_count(nT) % kResidentTiles;
  int64_t S = 1;
  while (S < 16 && Q * S * 2 <= kResidentTiles && nkb % (4 * S) == 0) S *= 2;
  *q = (Q > 0 && S >= 4) ? Q : 0;
  *split = *q > 0 ? S : 1;
}

// Shares of Q tiles over one round of workgroups: as many each as the round
// takes, at most `most`, of at least 4 staged blocks (which the shares need not
// divide evenly). 1 if the tiles are better left whole: the splits are parked and
// one more launch sums and finishes the tiles, which costs `cost_us`, so it has to
// save that. A staged block of 16 features takes a workgroup alone on its CU
// about 1.8 us in fp64 and 0.5 us in fp32, and a tile's splits are summed one
// after the other, about 0.6 of a block each, so no more than sqrt(nkb / 0.6) pay:
// the training at 502 x 2877 fp64 took 1.16 ms with 45 shares and takes 0.78 with
// 17, 561 x 1207 fp32 0.50 and 0.41.
//
// Beyond 256 shares some CUs take two, which share its matrix cores. In fp64 those
// are busy with one workgroup already and the launch waits for the CUs with two,
// 3.3 us per block; in fp32 a block takes up to 0.9 us as more CUs have two.
// Trainings whole and so shared: fp64 2800 x 260 (253 tiles, 506 shares) 1.54 and
// 2.05 ms, 2040 x 200 (136, 408) 1.30 and 1.57, 2800 x 1200 3.20 and 3.35, but 2040
// x 420 1.66 and 1.59, 2800 x 2000 4.93 and 4.77; fp32 2800 x 800 0.65 and 0.71, 2800
// x 1200 0.75 and 0.78, but 2200 x 1200 (171, 342) 0.75 and 0.70, 2040 x 800 0.54 and
// 0.50, 2800 x 2000 1.06 and 1.04.
inline int64_t share_tiles(int64_t Q, int64_t nkb, int64_t most, bool fp64, double cost_us,
                           int64_t* blocks) {
  *blocks = nkb;
  most = std::min(most, (int64_t)std::sqrt((double)nkb / 0.6));
  const int64_t want = std::min(std::min(kResidentTiles / Q, most), nkb / 4);
  if (want < 2) return 1;
  const int64_t per = round_up((nkb + want - 1) / want, 2), S = (nkb + per - 1) / per;
  const double block_us = fp64 ? 1.8 : 0.5, whole = (double)nkb * block_us;
  if (S < 2 || whole - (double)per * block_us < cost_us) return 1;
  if (Q * S > kCUs) {
    const double two = (double)(Q * S - kCUs) / kCUs;   // of the CUs
    const double each = fp64 ? 3.32 : block_us + 0.38 * two;
    if (whole - (double)per * each < (fp64 ? cost_us + 2.0 : 7.0)) return 1;
  }
  *blocks = per;
  return S;
}

// Which tiles of the polynomial and RBF kernels' products are split.
// - Few tiles (at most one per CU) leave most of the chip idle: all of them.
//   Trainings, whole and split: 502 x 2877 fp64 RBF 4.09 and 0.78 ms, 907 x 1100
//   2.50 and 1.10, 561 x 1207 fp32 cubic 1.00 and 0.41, 1500 x 2000 fp32 RBF 1.47
//   and 0.97.
// - Tiles left after the last full round of two per CU: tail_plan.
// - Otherwise those left after the last full round of one per CU, where they are
//   at most two thirds of one, in fp64: the CUs that take one more tile than the
//   others would run alone. A product: 5003 x 777 cubic (52 of 820 tiles) 0.407 and
//   0.375 ms, 3000 x 1000 RBF (44 of 300) 0.260 and 0.212, 4500 x 1500 (154 of 666)
//   0.586 and 0.560. The same in fp32, whose tiles are shorter, changed nothing
//   (3000 x 4000 0.260 and 0.262, 4358 x 1110 0.134 and 0.132).
inline void part_plan(int64_t W, int64_t tail_q, int64_t tail_split, int64_t nkb, bool fp64,
                      int64_t* q, int64_t* split, int64_t* blocks) {
  *q = 0;
  *split = 1;
  *blocks = nkb;
  if (W < 1) return;
  if (W <= kCUs) {
    *split = share_tiles(W, nkb, 64, fp64, 12.0, blocks);
    *q = *split > 1 ? W : 0;
  } else if (tail_q > 0) {
    *q = tail_q;
    *split = tail_split;
    *blocks = nkb / tail_split;
  } else if (fp64 && W % kCUs > 0 && W % kCUs <= kResidentTiles / 3) {
    *split = share_tiles(W % kCUs, nkb, 16, fp64, 24.0, blocks);
    *q = *split > 1 ? W % kCUs : 0;
  }
}

template <typename T>
Geometry geometry(int64_t n, int64_t d) {
  Geometry g{};
  g.n = n;
  g.d = d;
  g.N = n - 1;
  g.tile = TileShape<T>::T;
  g.bk = TileShape<T>::BK;
  g.ld = round_up(n, g.tile);
  g.nT = (g.N + g.tile - 1) / g.tile;
  g.NP = g.nT * g.tile;
  g.nb = cg_blocks(g.NP);
  g.plan_nkb = round_up(d, 2 * g.bk) / g.bk;
  tail_plan(g.nT, g.plan_nkb, &g.tail_q, &g.tail_split);
  // An even number of staged blocks (two LDS stages), as many as planned where
  // a plan shares them out: in fp32, whose staged blocks are half a planned
  // one, that can be 32 features of padding more.
  const int64_t W = tri_count(g.nT);
  const bool shared = (g.tail_q > 0 && W > kCUs) || g.NP <= kFusedMaxLinear;
  g.d_pad = shared ? g.plan_nkb * g.bk : round_up(d, 2 * TileShape<T>::SB);
  part_plan(W, g.tail_q, g.tail_split, g.d_pad / TileShape<T>::SB, sizeof(T) == 8,
            &g.part_q, &g.part_split, &g.part_blocks);
  return g;
}

// Carves aligned sub-buffers out of the caller's workspace (or only sizes them).
struct Carver {
  char* base;
  size_t off = 0;
  explicit Carver(void* b) : base(static_cast<char*>(b)) {}
  template <typename U>
  U* take(int64_t count) {
    U* p = base ? reinterpret_cast<U*>(base + off) : nullptr;
    off = align_up(off + (size_t)count * sizeof(U));
    return p;
  }
};

template <typename T>
struct TrainWs {
  store_t<T>* Xt;
  T* norms;
  double* q64;
  int64_t* acc; // fixed-point row sums of a product (two words per row)
  T* gpart;     // parked inner products of split tail tiles
  double* pq;   // per tile panel: sum p_j, then sum q_j p_j (2 nT)
  double *rhs, *x, *r, *dir, *qv;
  double* dir2;    // linear passes: the other buffer of the direction
  double *lin_part, *lin_w;   // linear passes: partial and whole w = X^T p
  double* xbest;   // iterate of the smallest recomputed residual (returned on a stall)
  double *bp0, *bp1, *bp2;
  double* scal;
  int* flags;
  uint32_t* order;
  double* hist;
  unsigned* ticket;   // workgroups done in a fused iteration's launch
  // what the stored points' inner products are multiplied by
  T gscale = T(1) / (T)(int64_t(1) << (2 * kStoredUp<T>));
  size_t bytes;
};


template <typename T>
TrainWs<T> carve_train(const Geometry& g, void* base) {
  Carver c(base);
  TrainWs<T> w{};
  w.Xt = c.take<store_t<T>>(TileShape<T>::SLICES * g.d_pad * g.ld);
  w.norms = c.take<T>(g.ld);
  w.q64 = c.take<double>(g.ld);
  // Row sums: two 64-bit words per row, however many tiles add to them; the
  // split tail's parked inner products (at most a quarter round of tiles).
  w.acc = c.take<int64_t>(2 * g.NP);
  w.gpart = c.take<T>(g.part_q * g.part_split * g.tile * g.tile);
  const int64_t chunks = lin_max_chunks(g.n, g.d);
  w.pq = c.take<double>(2 * std::max(g.nT, chunks));
  w.rhs = c.take<double>(g.NP);
  w.x = c.take<double>(g.NP);
  w.r = c.take<double>(g.NP);
  w.dir = c.take<double>(g.NP);
  w.qv = c.take<double>(g.NP);
  w.dir2 = c.take<double>(g.NP);
  w.lin_part = c.take<double>(2 * chunks * g.d);
  w.lin_w = c.take<double>(2 * g.d);
  w.xbest = c.take<double>(g.NP);
  w.bp0 = c.take<double>(kVecBlocks + 1);
  w.bp1 = c.take<double>(kVecBlocks + 1);
  w.bp2 = c.take<double>(kVecBlocks + 1);   // energy partials at residual recomputations
  w.scal = c.take<double>(S_COUNT);
  w.flags = c.take<int>(F_COUNT);
  w.order = c.take<uint32_t>(LSSVM_TILE_GROUP > 0 ? tri_count(g.nT) : 0);
  w.hist = c.take<double>(g.NP + 1);   // r^T r after each iteration (at most N of them)
  w.ticket = c.take<unsigned>(64);
  w.bytes = c.off;
  return w;
}

template <typename T>
struct PredictWs {
  store_t<T> *Xtr, *Xte;
  T *ntr, *nte, *alpha;
  double* part;
  int* flags;
  double* wait;      // nonzero while the scores wait for another layout
  double* few_part;  // few test points (over the layouts): partial scores, and whether
  int* few_bad;      // a workgroup met a value that is not finite
  double* lin_part;  // linear kernel: partial sums of w over point chunks
  double* lin_w;     // linear kernel: w = sum_i alpha_i x_i
  double* lin_f;     // linear kernel: <w, x> per test point
  int64_t ld_te, nTc, nTr;
  size_t bytes;
};

template <typename T>
PredictWs<T> carve_predict(const Geometry& g, int64_t n_test, void* base) {
  Carver c(base);
  PredictWs<T> w{};
  w.ld_te = round_up(n_test, g.tile);
  w.nTc = g.ld / g.tile;
  w.nTr = w.ld_te / g.tile;
  w.Xtr = c.take<store_t<T>>(TileShape<T>::SLICES * g.d_pad * g.ld);
  w.ntr = c.take<T>(g.ld);
  w.alpha = c.take<T>(g.ld);
  w.Xte = c.take<store_t<T>>(TileShape<T>::SLICES * g.d_pad * w.ld_te);
  w.nte = c.take<T>(w.ld_te);
  w.part = c.take<double>(w.nTc * w.ld_te);
  w.flags = c.take<int>(F_COUNT);
  w.wait = c.take<double>(1);
  w.lin_part = c.take<double>(2 * lin_max_chunks(g.n, g.d) * g.d);
  w.lin_w = c.take<double>(2 * g.d);
  w.lin_f = c.take<double>(n_test);
  w.bytes = c.off;
  if (n_test <= kFewTests) {
    // in place of the layouts, which few points do not use: at most 34 bytes per
    // model point, where a panel of the model takes 192 or more, so the size does
    // not depend on the path and never falls as n_test grows
    Carver f(base);
    const int64_t slots = predict_few_slots(g.n, n_test);
    w.few_part = f.take<double>(slots * n_test);
    w.few_bad = f.take<int>(slots);
    w.bytes = std::max(w.bytes, f.off);
  }
  return w;
}

// Host-side state of one call in flight: a pinned buffer for the few
// scalars read back per batch of CG iterations, and timing events (creating
// a few hundred events costs more than a small training takes). Calls lease
// a context from a process-wide pool and return it when they end, so the
// pool holds as many contexts as calls ever ran at once, however many
// threads come and go; contexts live until the process ends.
struct HostCtx {
  double* p = nullptr;   // 64 doubles, pinned
  int* flags = nullptr;  // inside p
  int device = -1;       // device the events belong to
  std::vector<hipEvent_t> ev;
  hipError_t ensure() {
    if (p) return hipSuccess;
    void* v = nullptr;
    hipError_t e = hipHostMalloc(&v, 64 * sizeof(double),
                                 hipHostMallocPortable | hipHostMallocMapped);
    if (e != hipSuccess) return e;
    p = static_cast<double*>(v);
    flags = reinterpret_cast<int*>(p + 32);
    return hipSuccess;
  }
};
std::mutex g_pool_mu;
std::vector<HostCtx*> g_pool_free;
std::atomic<int64_t> g_pool_size{0};
thread_local HostCtx* g_ctx = nullptr;   // the context of this thread's call in flight

struct CtxLease {
  HostCtx* prev;
  CtxLease() : prev(g_ctx) {
    std::lock_guard<std::mutex> lock(g_pool_mu);
    if (!g_pool_free.empty()) {
      g_ctx = g_pool_free.back();
      g_pool_free.pop_back();
    } else {
      g_ctx = new HostCtx();
      ++g_pool_size;
    }
  }
  ~CtxLease() {
    std::lock_guard<std::mutex> lock(g_pool_mu);
    g_pool_free.push_back(g_ctx);
    g_ctx = prev;
  }
  CtxLease(const CtxLease&) = delete;
  CtxLease& operator=(const CtxLease&) = delete;
};

// The input flags into g_ctx->flags, once the stream has been waited for.
hipError_t read_flags(const int* flags, hipStream_t s) {
  static_assert(F_COUNT * sizeof(int) == 2 * sizeof(double), "the flags are two words");
  return launch_read_back(reinterpret_cast<const double*>(flags), 2,
                          reinterpret_cast<double*>(g_ctx->flags), s);
}

// HIP events around each implicit product, recorded on the launch stream.
// Pairs carry the CG iteration they belong to, so products that ran after
// the stop (and returned at once) are left out.
struct MatvecTimer {
  static constexpr int kPairs = 2 * 64;   // up to two products per queued iteration
  bool on = false;
  hipEvent_t* ev = nullptr;   // 2 kPairs events of the thread's pool
  int64_t tag[kPairs] = {};
  int used = 0;          // event pairs recorded since the last harvest
  double total_ms = 0.0;
  int64_t count = 0;
  double* out = nullptr;   // caller's array of per-product times, or null
  int64_t cap = 0;
  hipError_t init(bool enable, double* times = nullptr, int64_t capacity = 0) {
    on = enable;
    out = times;
    cap = capacity;
    if (!on) return hipSuccess;
    int device = 0;
    hipError_t r = hipGetDevice(&device);
    if (r != hipSuccess) return r;
    HostCtx& c = *g_ctx;
    if (c.device != device) {
      for (hipEvent_t e : c.ev) (void)hipEventDestroy(e);
      c.ev.clear();
      c.device = device;
    }
    while (c.ev.size() < (size_t)(2 * kPairs)) {
      hipEvent_t e = nullptr;
      if ((r = hipEventCreate(&e)) != hipSuccess) return r;
      c.ev.push_back(e);
    }
    ev = c.ev.data();
    return hipSuccess;
  }
  // A batch queues at most 32 iterations of at most two products each, so the
  // pairs never run out; should they, the extra products are simply not timed.
  bool full() const { return used >= kPairs; }
  hipError_t start(hipStream_t s, int64_t iter) {
    if (!on || full()) return hipSuccess;
    tag[used] = iter;
    return hipEventRecord(ev[2 * used], s);
  }
  hipError_t stop(hipStream_t s) {
    if (!on || full()) return hipSuccess;
    hipError_t r = hipEventRecord(ev[2 * used + 1], s);
    ++used;
    return r;
  }
  // After the stream has been synchronised: add the pairs of iterations <= last.
  hipError_t harvest(int64_t last) {
    for (int i = 0; i < used; ++i) {
      if (tag[i] > last) continue;
      float ms = 0.f;
      hipError_t r = hipEventElapsedTime(&ms, ev[2 * i], ev[2 * i + 1]);
      if (r != hipSuccess) return r;
      total_ms += ms;
      if (out && count < cap) out[count] = ms;
      ++count;
    }
    used = 0;
    return hipSuccess;
  }
};

bool valid_dtype(int32_t dt) { return dt == LSSVM_F64 || dt == LSSVM_F32; }
bool valid_kernel(int32_t k) { return k == LSSVM_LINEAR || k == LSSVM_POLY || k == LSSVM_RBF; }

int check_kernel_params(int32_t kernel, const lssvm_params* kp) {
  if (!valid_kernel(kernel)) return fail(LSSVM_EINVAL, "unknown kernel %d", (int)kernel);
  if (kernel == LSSVM_LINEAR) return LSSVM_OK;
  if (!kp) return fail(LSSVM_EINVAL, "kernel parameters required for kernel %d", (int)kernel);
  if (!(kp->gamma > 0.0) || !std::isfinite(kp->gamma))
    return fail(LSSVM_EINVAL, "gamma must be finite and > 0 (got %g)", kp->gamma);
  if (kernel == LSSVM_POLY) {
    if (kp->degree < 1) return fail(LSSVM_EINVAL, "degree must be >= 1 (got %d)", kp->degree);
    if (!std::isfinite(kp->coef0)) return fail(LSSVM_EINVAL, "coef0 must be finite");
  }
  return LSSVM_OK;
}

int check_sizes(int64_t n, int64_t d, int64_t min_n) {
  if (n < min_n) return fail(LSSVM_EINVAL, "n must be >= %lld (got %lld)", (long long)min_n,
                             (long long)n);
  if (d < 1) return fail(LSSVM_EINVAL, "d must be >= 1 (got %lld)", (long long)d);
  if (n > kMaxPoints || d > kMaxFeatures)
    return fail(LSSVM_EINVAL, "problem too large (n=%lld, d=%lld)", (long long)n, (long long)d);
  return LSSVM_OK;
}

int check_workspace(const void* ws, size_t have, size_t need) {
  if (!ws) return fail(LSSVM_EINVAL, "workspace is NULL");
  if (reinterpret_cast<uintptr_t>(ws) % kAlign != 0)
    return fail(LSSVM_EINVAL, "workspace must be %zu-byte aligned", kAlign);
  if (have < need)
    return fail(LSSVM_EINVAL, "workspace too small: %zu bytes given, %zu needed", have, need);
  return LSSVM_OK;
}

// Exponent scale of the RBF tile epilogue: fp32 evaluates exp(-gamma dist)
// as exp2(-(gamma log2 e) dist) on the hardware base-2 exponential.
template <typename T> T rbf_scale(double gamma);
template <> float rbf_scale<float>(double gamma) { return (float)(gamma * 1.4426950408889634); }
template <> double rbf_scale<double>(double gamma) { return gamma; }

// Workgroups per tile of every product of n points (a training's CG
// iterations, its residual recomputations, a warm start's and the true
// residual's products, lssvm_matvec) on whole tiles. The linear kernel has tiles
// only on small problems, whose iterations are fused launches: the few tiles take
// one CU each and their matrix work is most of the launch, so their features are
// split as far as one round of workgroups allows, down to a single feature block
// per workgroup.
// All products of a problem take the same split: each split rounds the
// operator its own way (fp32 partial inner products), and a recomputed
// residual from a differently rounded operator than the iterations' stalls
// fp32 CG above its eps.
inline int64_t product_split(const Geometry& g, int32_t kernel) {
  if (kernel != LSSVM_LINEAR) return 1;
  int64_t S = 1;
  const int64_t nkb = g.plan_nkb, W = tri_count(g.nT);
  // double while every workgroup keeps an even block count (the two-stage
  // loop) or gets exactly one (the single-block variant)
  while (S < LSSVM_LINEAR_SPLIT_MAX && W * 2 * S <= kResidentTiles &&
         (nkb % (4 * S) == 0 || nkb == 2 * S))
    S *= 2;
  return S;
}

template <typename T>
TileArgs<T> sym_args(const Geometry& g, const TrainWs<T>& w, const lssvm_params& kp,
                     int32_t kernel, const double* p) {
  TileArgs<T> a{};
  a.A = w.Xt;
  a.B = w.Xt;
  a.nkb = g.d_pad / TileShape<T>::SB;
  a.nA = w.norms;
  a.nB = w.norms;
  a.pv = p;
  a.q64 = w.q64;
  a.pq = w.pq;
  a.gscale = w.gscale;
  a.gamma = (T)kp.gamma;
  a.coef0 = (T)kp.coef0;
  a.gamma64 = kp.gamma;
  a.coef64 = kp.coef0;
  a.rbf_scale = rbf_scale<T>(kp.gamma);
  a.degree = kp.degree;
  a.nTc = g.nT;
  a.ksplit = product_split(g, kernel);
  a.split_blocks = a.nkb / a.ksplit;
  a.order = LSSVM_TILE_GROUP > 0 ? w.order : nullptr;
  a.acc = w.acc;
  a.fx = w.scal + S_PMAX;      // [S_PMAX], [S_NMAX], [S_FIXSC]
  a.fx_bad = w.flags + F_PRODUCT;
  return a;
}

// The tile visit order, written into the workspace on the device (once per
// call); the same launch zeroes the flags, the scalars and the row-sum words.
template <typename T>
int clear_and_order(const Geometry& g, const TrainWs<T>& w, hipStream_t s) {
  const bool ordered = LSSVM_TILE_GROUP > 0 && g.nT > 0;
  LSSVM_HIP(launch_setup_clear(g.nT, LSSVM_TILE_GROUP, ordered ? w.order : nullptr, w.flags,
                               w.scal, w.acc, 2 * g.NP, w.ticket, s));
  return LSSVM_OK;
}

// fp32 points with values that the usual scale does not serve (F_RANGE, raised by the
// layout kernel) are laid out again, multiplied by 2^up so that their largest value is
// about 2^52, whose products (2^104, times 2^21 features) still fit. up stays below
// 64, for 2^-2up to be a float, and at 0 for larger values, whose products may not fit
// as they are. (Beside values above 2^40, products more than 2^206 below the square of
// the largest lose bits that fp32 would hold.) Rare, so it may wait for the device. The
// flag is down afterwards.
int relayout(const float* X, int64_t n, int64_t d, uint16_t* Xt, int64_t ld, int64_t d_pad,
             int* flags, int* up, hipStream_t s) {
  int* word = flags + F_RANGE;
  LSSVM_HIP(hipMemsetAsync(word, 0, sizeof(int), s));
  LSSVM_HIP(launch_abs_max(X, n * d, word, s));
  LSSVM_HIP(hipMemcpyAsync(g_ctx->flags, word, sizeof(int), hipMemcpyDeviceToHost, s));
  LSSVM_HIP(hipStreamSynchronize(s));
  float top;
  std::memcpy(&top, g_ctx->flags, sizeof top);
  *up = std::min(63, std::max(0, 52 - (top > 0.f ? std::ilogb(top) : 0)));
  LSSVM_HIP(hipMemsetAsync(word, 0, sizeof(int), s));
  LSSVM_HIP(launch_layout<float>(X, n, d, Xt, ld, d_pad, *up, 0, flags, s));
  return LSSVM_OK;
}
int relayout(const double*, int64_t, int64_t, double*, int64_t, int64_t, int*, int*,
             hipStream_t) {
  return LSSVM_OK;   // fp64 points are stored as they are
}

// Norms, q and k_mm of the training points as they lie in the layout.
template <typename T>
int setup_norms(const Geometry& g, const TrainWs<T>& w, int up, int32_t kernel,
                const lssvm_params& kp, hipStream_t s) {
  LSSVM_HIP(launch_norms_q<T>(w.Xt, g.ld, g.d_pad, g.N, g.N, up, kernel, kp.gamma, kp.coef0,
                              kp.degree, w.norms, w.q64, w.scal, s));
  return LSSVM_OK;
}

// The training points, rows and columns of every product, laid out by their range;
// what the first layout's norms and q overflowed in is formed again.
template <typename T>
int rescale_points(const Geometry& g, TrainWs<T>& w, const T* X, int32_t kernel,
                   const lssvm_params& kp, hipStream_t s) {
  int up = 0;
  LSSVM_TRY(relayout(X, g.n, g.d, w.Xt, g.ld, g.d_pad, w.flags, &up, s));
  w.gscale = (T)std::ldexp(1.0, -2 * up);
  LSSVM_HIP(hipMemsetAsync(w.scal + S_NMAX, 0, sizeof(double), s));
  return setup_norms<T>(g, w, up, kernel, kp, s);
}

// a1 + a2: layout, norms, q and k_mm, left on the device. The caller reads the
// input flags back with its result: a non-finite X is an error, and points out of the
// usual range are laid out again.
template <typename T>
int setup_points(const Geometry& g, const TrainWs<T>& w, const T* X, int32_t kernel,
                 const lssvm_params& kp, hipStream_t s) {
  LSSVM_TRY(clear_and_order<T>(g, w, s));
  LSSVM_HIP(launch_layout<T>(X, g.n, g.d, w.Xt, g.ld, g.d_pad, kStoredUp<T>, 1, w.flags, s));
  return setup_norms<T>(g, w, kStoredUp<T>, kernel, kp, s);
}

// A finished product's row sums and the terms of Q~ p the tiles leave out.
template <typename T>
RankOne rank_one(const Geometry& g, const TrainWs<T>& w, int32_t kernel, double C,
                 const double* p) {
  (void)kernel;
  return RankOne{w.pq, g.nT, w.acc, w.q64, p, w.scal, w.flags, 1.0 / C, nullptr};
}

// The linear kernel's two passes over the caller's points.
template <typename T>
struct LinearPasses {
  const Geometry& g;
  const TrainWs<T>& w;
  const T* X;
  double C;
  hipStream_t s;
  int64_t nch, nbg;   // chunks of w; block partials of a gather
  LinearPasses(const Geometry& g_, const TrainWs<T>& w_, const T* X_, double C_, hipStream_t s_)
      : g(g_), w(w_), X(X_), C(C_), s(s_), nch(lin_shape(g_.N, g_.d, lin_vec(X_, g_.d)).nch),
        nbg(lin_gather_blocks(X_, g_.N, g_.d)) {}
  RankOne rank_one(const double* p, const double* kp) const {
    return RankOne{w.pq, nch, nullptr, w.q64, p, w.scal, w.flags, 1.0 / C, kp};
  }
  // w = X^T p, with S and T of p
  hipError_t weights(const LinVec& v) const {
    return launch_lin_w<T>(X, g.N, g.d, v, w.q64, w.lin_part, w.lin_w, w.pq, s);
  }
  LinVec vec(const double* p, bool stop) const {
    LinVec v{};
    v.p = p;
    v.scal = w.scal;
    v.stop = stop;
    return v;
  }
  // K p into qv, for the readers of rank_one(p, qv)
  int product(const double* p, bool stop) const {
    LSSVM_HIP(weights(vec(p, stop)));
    LSSVM_HIP(launch_lin_kp<T>(X, g.N, g.d, w.lin_w, w.qv, s));
    return LSSVM_OK;
  }
};

// The first of the two launches of a product's split tiles: parks their inner
// products, and leaves a as the second, the fixup, takes it.
template <typename T>
hipError_t launch_parked(const Geometry& g, TileArgs<T>& a, int32_t kernel, T* gpart,
                         hipStream_t s) {
  a.tile_offset = tri_count(g.nT) - g.part_q;
  a.ksplit = g.part_split;
  a.split_blocks = g.part_blocks;
  a.gpart = gpart;
  return launch_tiles_sym<T>(a, kernel, kPartial, g.part_q * g.part_split, s);
}

// The tile launches of one product: all tiles whole (the linear kernel's split
// tiles included) but the last part_q, which are split, parked and fixed up.
template <typename T>
hipError_t launch_product(const Geometry& g, TileArgs<T> a, int32_t kernel, T* gpart,
                          hipStream_t s) {
  const int64_t W = tri_count(g.nT);
  if (kernel == LSSVM_LINEAR) return launch_tiles_sym<T>(a, kernel, kWhole, W * a.ksplit, s);
  if (g.part_q < W) {
    const hipError_t e = launch_tiles_sym<T>(a, kernel, kWhole, W - g.part_q, s);
    if (e != hipSuccess || g.part_q == 0) return e;
  }
  const hipError_t e = launch_parked<T>(g, a, kernel, gpart, s);
  if (e != hipSuccess) return e;
  return launch_tiles_sym<T>(a, kernel, kFixup, g.part_q, s);
}

// One implicit product K p into the partial-sum buffer (plus the per-panel
// sums of the rank-one terms).
template <typename T>
int matvec_partials(const Geometry& g, const TrainWs<T>& w, const lssvm_params& kp,
                    int32_t kernel, const double* p, hipStream_t s) {
  LSSVM_HIP(launch_product<T>(g, sym_args<T>(g, w, kp, kernel, p), kernel, w.gpart, s));
  return LSSVM_OK;
}

template <typename T>
int timed_matvec(const Geometry& g, const TrainWs<T>& w, const lssvm_params& kp, int32_t kernel,
                 const double* p, hipStream_t s, MatvecTimer& tm, int64_t iter) {
  LSSVM_HIP(tm.start(s, iter));
  TileArgs<T> a = sym_args<T>(g, w, kp, kernel, p);
  a.stop = w.scal + S_STATUS + ST_DONE;   // skip the launches once CG has stopped
  LSSVM_HIP(launch_product<T>(g, a, kernel, w.gpart, s));
  LSSVM_HIP(tm.stop(s));
  return LSSVM_OK;
}


// How CG ended, for the report.
struct CgEnd {
  int64_t it = 0, extra_products = 0, n_timed = 0;
  bool converged = false, broke = false, stalled = false;
  double delta0 = 0.0, delta = 0.0, t_setup = 0.0, t_cg = 0.0, t_matvec = 0.0;
  int status = LSSVM_OK;
  double rel() const { return delta0 > 0.0 ? std::sqrt(delta / delta0) : 0.0; }
};

void fill_info(const CgEnd& e, lssvm_info* info, double t_total) {
  if (!info) return;
  info->iterations = e.it;
  info->stop_reason = e.broke     ? LSSVM_STOP_BREAKDOWN
                      : e.stalled ? LSSVM_STOP_STALL
                      : e.converged ? LSSVM_STOP_EPS
                                    : LSSVM_STOP_MAX_ITER;
  info->rel_residual = e.rel();
  // products: one per iteration plus each completed residual recomputation
  // (a breakdown stops before its iteration's recomputation)
  info->n_matvec = e.it + (e.broke ? e.it - 1 : e.it) / kReplaceEvery + e.extra_products;
  info->t_matvec_ms = e.t_matvec;
  info->n_matvec_timed = e.n_timed;
  info->t_setup_ms = e.t_setup;
  info->t_cg_ms = e.t_cg;
  info->t_total_ms = t_total;
}

// The end of CG: its message and status, the residual history. A breakdown
// leaves the outputs untouched, and the report says how far CG got.
template <typename T>
int end_cg(const Geometry& g, const TrainWs<T>& w, CgEnd& e, int status, lssvm_info* info,
           clock_t_::time_point t0, hipStream_t s) {
  if (status < 0) {
    fill_info(e, info, ms_since(t0));
    return status;
  }
  if (e.stalled)
    e.status = fail(LSSVM_NOT_CONVERGED,
                    "CG stalled after %lld iterations: no new minimum of the true residual or the "
                    "energy (best relative residual %g)", (long long)e.it, e.rel());
  else if (!e.converged)
    e.status = fail(LSSVM_NOT_CONVERGED, "CG stopped after %lld iterations at relative residual %g",
                    (long long)e.it, e.rel());
  if (info && info->residual_history && e.it > 0) {
    const int64_t nh = std::min(std::min(e.it, info->history_capacity), g.NP + 1);
    if (nh > 0) {
      LSSVM_HIP(hipMemcpyAsync(info->residual_history, w.hist, nh * sizeof(double),
                               hipMemcpyDeviceToHost, s));
      LSSVM_HIP(hipStreamSynchronize(s));
      for (int64_t k = 0; k < nh; ++k) info->residual_history[k] /= e.delta0;
    }
  }
  return LSSVM_OK;
}

// The report of a finished training (the optional true-residual product, which
// follows, is not training).
void end_report(const Geometry& g, const CgEnd& e, lssvm_info* info, clock_t_::time_point t0) {
  const double t_total = ms_since(t0);
  if (log_enabled())
    std::fprintf(stderr,
                 "[lssvm] train n=%lld d=%lld: %lld iterations, relative residual %.3e, "
                 "setup %.2f ms, cg %.2f ms, total %.2f ms\n",
                 (long long)g.n, (long long)g.d, (long long)e.it, e.rel(), e.t_setup, e.t_cg,
                 t_total);
  fill_info(e, info, t_total);
}

// info->true_rel_residual from a finished product of x.
template <typename T>
int true_residual(const Geometry& g, const TrainWs<T>& w, const RankOne& c, int64_t NP,
                  double delta0, lssvm_info* info, hipStream_t s) {
  double tr = 0.0;
  if (delta0 > 0.0) {
    LSSVM_HIP(launch_true_residual(c, NP, g.N, w.rhs, w.bp1, s));
    LSSVM_HIP(launch_finish_sum(w.bp1, cg_blocks(NP), w.scal, S_TRUE, s));
    LSSVM_HIP(hipMemcpyAsync(g_ctx->p, w.scal + S_TRUE, sizeof(double), hipMemcpyDeviceToHost, s));
    LSSVM_HIP(hipStreamSynchronize(s));
    tr = std::sqrt(g_ctx->p[0] / delta0);
  }
  info->true_rel_residual = tr;
  return LSSVM_OK;
}

// A whole linear training in one launch and one read-back (k_lin_train).
template <typename T>
int train_small_linear(const Geometry& g, const TrainWs<T>& w, const T* X, const T* y, double C,
                       double eps, int64_t max_iter, T* alpha_out, double* b_out, lssvm_info* info,
                       clock_t_::time_point t0, hipStream_t s) {
  LinTrain a{};
  a.invC = 1.0 / C;
  a.eps2 = eps * eps;
  a.max_iter = (int)std::min<int64_t>(max_iter > 0 ? max_iter : g.N, INT32_MAX);
  a.replace_every = (int)kReplaceEvery;
  a.x = w.x;
  a.rhs = w.rhs;
  a.q64 = w.q64;
  a.scal = w.scal;
  a.hist = w.hist;
  a.hist_cap = g.NP + 1;
  a.flags = w.flags;
  LSSVM_HIP(launch_lin_train<T>(X, y, g.n, g.d, a, alpha_out, s));
  LSSVM_HIP(launch_read_back(w.scal, S_COUNT, g_ctx->p, s));
  LSSVM_HIP(hipStreamSynchronize(s));
  const double* p = g_ctx->p;
  const double* st = p + S_STATUS;
  const int inflags = (int)p[S_INFLAGS];
  if (inflags & 1) return fail(LSSVM_ENONFINITE, "X holds a NaN or an infinity");
  if (inflags & 2) return fail(LSSVM_EBADLABEL, "labels must be +1 or -1");
  constexpr double kTicksPerMs = 1e5;   // the device's wall clock runs at 100 MHz
  CgEnd e;
  e.broke = st[ST_BREAK] != 0.0;
  e.stalled = st[ST_STALL] != 0.0;
  e.converged = st[ST_DONE] != 0.0 && !e.broke && !e.stalled;
  e.it = (int64_t)st[ST_ITER] + (e.broke ? 1 : 0);   // the update of the next found the curvature
  e.delta0 = p[S_DELTA0];
  e.delta = st[ST_DELTA];
  e.t_setup = p[S_TIMES] / kTicksPerMs;
  e.t_cg = p[S_TIMES + 1] / kTicksPerMs;
  const double b = p[S_B];
  int status = LSSVM_OK;
  if (e.broke)
    status = fail(LSSVM_EBREAKDOWN, "CG breakdown at iteration %lld (d^T Q d = %g)",
                  (long long)e.it, st[ST_CURV]);
  LSSVM_TRY(end_cg<T>(g, w, e, status, info, t0, s));
  *b_out = b;
  end_report(g, e, info, t0);
  if (info && info->compute_true_residual) {
    const LinearPasses<T> lin(g, w, X, C, s);
    if (e.delta0 > 0.0) LSSVM_TRY(lin.product(w.x, false));
    LSSVM_TRY(true_residual<T>(g, w, lin.rank_one(w.x, w.qv), g.N, e.delta0, info, s));
  }
  return e.status;
}

template <typename T>
int train_impl(const T* X, const T* y, int64_t n, int64_t d, int32_t kernel,
               const lssvm_params& kp, double C, double eps, int64_t max_iter, void* workspace,
               size_t ws_bytes, T* alpha_out, double* b_out, lssvm_info* info, hipStream_t s) {
  const auto t0 = clock_t_::now();
  const Geometry g = geometry<T>(n, d);
  TrainWs<T> w = carve_train<T>(g, nullptr);
  LSSVM_TRY(check_workspace(workspace, ws_bytes, w.bytes));
  w = carve_train<T>(g, workspace);
  LSSVM_HIP(g_ctx->ensure());

  if (info) {
    info->iterations = 0;
    info->n_matvec = 0;
    info->t_matvec_ms = 0.0;
    info->n_matvec_timed = 0;
    info->rel_residual = 0.0;
    info->true_rel_residual = -1.0;
    info->t_setup_ms = info->t_cg_ms = info->t_total_ms = 0.0;
    info->stop_reason = LSSVM_STOP_EPS;
  }

  if (n == 1) {  // alpha = [0], b = y_0
    LSSVM_HIP(hipMemsetAsync(w.flags, 0, F_COUNT * sizeof(int), s));
    LSSVM_HIP(launch_layout<T>(X, g.n, g.d, w.Xt, g.ld, g.d_pad, kStoredUp<T>, 1, w.flags, s));
    LSSVM_HIP(launch_single_point<T>(y, alpha_out, w.scal, w.flags, s));
    LSSVM_HIP(read_flags(w.flags, s));
    LSSVM_HIP(hipMemcpyAsync(g_ctx->p, w.scal + S_B, sizeof(double), hipMemcpyDeviceToHost, s));
    LSSVM_HIP(hipStreamSynchronize(s));
    if (g_ctx->flags[F_NONFINITE]) return fail(LSSVM_ENONFINITE, "X holds a NaN or an infinity");
    if (g_ctx->flags[F_BADLABEL]) return fail(LSSVM_EBADLABEL, "labels must be +1 or -1");
    *b_out = g_ctx->p[0];
    if (info) {
      info->rel_residual = 0.0;
      info->true_rel_residual = info->compute_true_residual ? 0.0 : -1.0;
      info->t_total_ms = ms_since(t0);
    }
    return LSSVM_OK;
  }

  // A linear problem that fits one workgroup's LDS, from a zero start and with no
  // product timed on its own.
  if (kernel == LSSVM_LINEAR && lin_train_fits(n, d, sizeof(T)) &&
      !(info && (info->warm_start || info->time_matvec)))
    return train_small_linear<T>(g, w, X, y, C, eps, max_iter, alpha_out, b_out, info, t0, s);

  // ---- setup: a1, a2, a3 (one read-back for the input flags and r0^T r0)
  // Linear passes keep the points as they are and their vectors unpadded.
  const bool passes = linear_passes(g, kernel);
  const int64_t NP = passes ? g.N : g.NP, nb = cg_blocks(NP);
  const LinearPasses<T> lin(g, w, X, C, s);
  if (passes) {
    LSSVM_HIP(launch_setup_clear(0, LSSVM_TILE_GROUP, nullptr, w.flags, w.scal, nullptr, 0,
                                 nullptr, s));
    LSSVM_HIP(launch_lin_q<T>(X, g.n, g.d, w.q64, w.scal, w.flags, s));
  } else {
    LSSVM_TRY(setup_points<T>(g, w, X, kernel, kp, s));
  }
  LSSVM_HIP(launch_rhs_init<T>(y, g.N, NP, w.rhs, w.x, w.xbest, w.r, w.dir, w.bp0, w.flags,
                               w.scal, s));
  LSSVM_HIP(launch_finish_delta0(w.bp0, nb, w.scal, eps * eps, w.flags, s));
  // one read-back: r0^T r0 and the input flags
  LSSVM_HIP(launch_read_back(w.scal + S_DELTA0, S_INFLAGS - S_DELTA0 + 1, g_ctx->p, s));
  LSSVM_HIP(hipStreamSynchronize(s));
  const int inflags = (int)g_ctx->p[S_INFLAGS - S_DELTA0];
  if (inflags & 1) return fail(LSSVM_ENONFINITE, "X holds a NaN or an infinity");
  if (inflags & 2) return fail(LSSVM_EBADLABEL, "labels must be +1 or -1");
  const double delta0 = g_ctx->p[0];
  if (inflags & 4) LSSVM_TRY(rescale_points<T>(g, w, X, kernel, kp, s));
  const double t_setup = ms_since(t0);
  MatvecTimer tm;
  LSSVM_HIP(tm.init(info && info->time_matvec, info ? info->matvec_times : nullptr,
                    info ? info->matvec_times_capacity : 0));

  // ---- a4 + a5: conjugate gradients
  // Iterations are enqueued in batches (1, 2, 4, ... up to 32) and the status
  // is read once per batch; kernels queued after the stop return at once, so
  // the iterate is the one of the stopping iteration. CG stops on eps, on
  // curvature breakdown, or stalled: at a residual recomputation neither the
  // true residual nor the energy set a new minimum (the iterate is then the
  // one with the smallest recomputed residual).
  const auto t1 = clock_t_::now();
  if (max_iter <= 0) max_iter = g.N;
  int64_t queued = 0, it = 0;
  bool done = delta0 == 0.0;  // all labels equal: alpha~ = 0 solves the system
  bool broke = false, stalled = false;
  double delta = delta0;
  int status = LSSVM_OK;
  int64_t batch = 1;   // fused (small) problems start at 8, below
  double* st = g_ctx->p;
  int64_t extra_products = 0;
  constexpr int64_t kMaxBatch = 32;
  auto product_of = [&](const double* p) {   // a finished product, for its readers
    return passes ? lin.rank_one(p, w.qv) : rank_one(g, w, kernel, C, p);
  };
  if (info && info->warm_start && !done) {
    // x0 = the caller's alpha~, r0 = rhs - Q~ x0, dir = r0; the stop threshold
    // set from rhs^T rhs above is kept
    LSSVM_HIP(launch_pad_to_f64<T>(alpha_out, g.N, w.x, NP, w.scal, nullptr, s));
    if (passes) LSSVM_TRY(lin.product(w.x, false));
    else LSSVM_TRY(matvec_partials<T>(g, w, kp, kernel, w.x, s));
    LSSVM_HIP(launch_cg_residual(product_of(w.x), NP, g.N, w.rhs, w.r, w.bp1, w.bp2, s));
    LSSVM_HIP(launch_warm_start(w.bp1, w.bp2, nb, w.scal, w.r, w.dir, w.x, w.xbest, NP, s));
    LSSVM_HIP(launch_read_back(w.scal + S_STATUS, ST_COUNT, st, s));
    LSSVM_HIP(hipStreamSynchronize(s));
    delta = st[ST_DELTA];
    done = st[ST_DONE] != 0.0;
    extra_products = 1;
    if (!std::isfinite(delta))
      return fail(LSSVM_ENONFINITE, "the warm-start alpha gives a non-finite residual");
  }
  // Iterations queued after the stop return at once but still pay for their
  // launches, so once two status reads give a rate of decrease of r^T r, a
  // batch is also capped at the iterations that rate needs to reach the stop
  // threshold (with a quarter to spare).
  int64_t it_prev = 0, need = max_iter;
  double delta_prev = delta;
  const bool fused = !passes && fused_iteration(g, kernel);
  // A fused iteration takes ~15 us and a status read-back ~30 us: small
  // problems start with 8 iterations queued (those run past the stop return at
  // once, a few microseconds each)
  if (fused) batch = 8;
  // Linear passes form the direction of the next iteration with its product
  // (from one buffer into the other); `pending` until then. The last one of a
  // batch is formed on its own, so that the status is complete when read.
  double *dir = w.dir, *dir_other = w.dir2;
  bool pending = false;
  const bool trusted = !passes || eps >= kTrustedEps;
  double* dir_of[kMaxBatch];   // linear passes: the direction of each iteration of a batch
  while (!done && queued < max_iter) {
    const int64_t nq = std::min<int64_t>(std::min(batch, need), max_iter - queued);
    for (int64_t b = 0; b < nq; ++b) {
      const int64_t k = ++queued;
      const int par = (int)((k - 1) & 1);  // r^T r of the current iterate lives in S_DHIST + par
      const bool refresh = k % kReplaceEvery == 0;
      if (fused && !refresh) {   // product and vector work in one launch
        LSSVM_HIP(tm.start(s, k));
        TileArgs<T> a = sym_args<T>(g, w, kp, kernel, w.dir);
        a.stop = w.scal + S_STATUS + ST_DONE;
        FusedCg f{w.ticket, rank_one(g, w, kernel, C, w.dir), w.qv, w.x, w.r, w.dir, w.scal,
                  w.hist, g.NP, g.N, k, g.NP + 1, par};
        const int64_t W = tri_count(g.nT);
        const bool split = kernel != LSSVM_LINEAR && g.part_q > 0;   // all: few tiles
        if (split) LSSVM_HIP(launch_parked<T>(g, a, kernel, w.gpart, s));
        LSSVM_HIP(launch_tiles_cg<T>(a, kernel, split ? kFixup : kWhole,
                                     kernel == LSSVM_LINEAR ? W * a.ksplit : W, f, s));
        LSSVM_HIP(tm.stop(s));
        continue;
      }
      if (passes) {
        LSSVM_HIP(tm.start(s, k));
        LinVec v = lin.vec(dir, true);
        if (pending) {
          v.r = w.r;
          v.dir_out = dir_other;
          v.bp = w.bp1;
          v.nb = nb;
          v.par = par ^ 1;
          v.iter = k - 1;
          v.hist = w.hist;
          v.hist_cap = g.NP + 1;
          std::swap(dir, dir_other);
        }
        dir_of[b] = dir;
        LSSVM_HIP(lin.weights(v));
        LSSVM_HIP(launch_lin_gather<T>(X, g.N, g.d, w.lin_w, lin.rank_one(dir, nullptr), w.qv,
                                       w.bp0, s));
        LSSVM_HIP(tm.stop(s));
        LSSVM_HIP(launch_cg_update(refresh, w.bp0, lin.nbg, w.scal, par, dir, w.qv, w.x, w.r,
                                   w.bp1, NP, s));
        pending = true;
        if (refresh) {
          LSSVM_HIP(tm.start(s, k));
          LSSVM_TRY(lin.product(w.x, true));
          LSSVM_HIP(tm.stop(s));
          LSSVM_HIP(launch_cg_residual(product_of(w.x), NP, g.N, w.rhs, w.r, w.bp1, w.bp2, s));
        }
        if (refresh || b + 1 == nq) {
          LSSVM_HIP(launch_cg_direction(w.bp1, nb, w.scal, par, k, w.r, dir, NP, w.hist, g.NP + 1,
                                        refresh ? k / kReplaceEvery : 0, 0, w.bp2, w.x, w.xbest,
                                        s));
          pending = false;
        }
        continue;
      }
      LSSVM_TRY(timed_matvec<T>(g, w, kp, kernel, w.dir, s, tm, k));
      LSSVM_HIP(launch_cg_gather(rank_one(g, w, kernel, C, w.dir), g.NP, g.N, w.qv, w.bp0, s));
      if (refresh) {
        LSSVM_HIP(launch_cg_update(1, w.bp0, g.nb, w.scal, par, w.dir, w.qv, w.x, w.r, w.bp1,
                                   g.NP, s));
        LSSVM_TRY(timed_matvec<T>(g, w, kp, kernel, w.x, s, tm, k));
        LSSVM_HIP(launch_cg_residual(rank_one(g, w, kernel, C, w.x), g.NP, g.N, w.rhs,
                                     w.r, w.bp1, w.bp2, s));
      } else {
        LSSVM_HIP(launch_cg_update(0, w.bp0, g.nb, w.scal, par, w.dir, w.qv, w.x, w.r, w.bp1,
                                   g.NP, s));
      }
      LSSVM_HIP(launch_cg_direction(w.bp1, g.nb, w.scal, par, k, w.r, w.dir, g.NP, w.hist,
                                    g.NP + 1, refresh ? k / kReplaceEvery : 0, 1, w.bp2,
                                    w.x, w.xbest, s));
    }
    const int64_t first = queued - nq + 1;
    LSSVM_HIP(launch_read_back(w.scal + S_STATUS, ST_COUNT, st, s));
    LSSVM_HIP(hipStreamSynchronize(s));
    it = (int64_t)st[ST_ITER];
    done = st[ST_DONE] != 0.0;
    broke = st[ST_BREAK] != 0.0;
    stalled = st[ST_STALL] != 0.0;
    LSSVM_HIP(tm.harvest(done ? it : queued));
    if (broke) {
      it += 1;   // the update of the next iteration found the curvature
      status = fail(LSSVM_EBREAKDOWN, "CG breakdown at iteration %lld (d^T Q d = %g)",
                    (long long)it, st[ST_CURV]);
      break;
    }
    if (!trusted && done && !stalled && it % kReplaceEvery != 0 && it < max_iter) {
      // the recurrence met eps: the residual itself, and on from there if it does not
      dir = dir_of[it - first];
      dir_other = dir == w.dir ? w.dir2 : w.dir;
      queued = it;
      extra_products += 1;
      LSSVM_HIP(hipMemsetAsync(w.scal + S_STATUS + ST_DONE, 0, sizeof(double), s));
      LSSVM_HIP(tm.start(s, it));
      LSSVM_TRY(lin.product(w.x, false));
      LSSVM_HIP(tm.stop(s));
      LSSVM_HIP(launch_cg_residual(product_of(w.x), NP, g.N, w.rhs, w.r, w.bp1, w.bp2, s));
      LSSVM_HIP(launch_cg_direction(w.bp1, nb, w.scal, (int)((it - 1) & 1), it, w.r, dir, NP,
                                    w.hist, g.NP + 1, 0, 0, w.bp2, w.x, w.xbest, s));
      LSSVM_HIP(launch_read_back(w.scal + S_STATUS, ST_COUNT, st, s));
      LSSVM_HIP(hipStreamSynchronize(s));
      LSSVM_HIP(tm.harvest(it));
      done = st[ST_DONE] != 0.0;
    }
    delta = st[ST_DELTA];
    if (log_enabled())
      std::fprintf(stderr, "[lssvm] CG iteration %lld: relative residual %.3e (%.1f ms)\n",
                   (long long)it, delta0 > 0.0 ? std::sqrt(delta / delta0) : 0.0,
                   ms_since(t1));
    batch = std::min<int64_t>(2 * batch, kMaxBatch);
    need = max_iter;
    if (it > it_prev && delta > 0.0 && delta < delta_prev && st[ST_STOP] < delta) {
      const double per_it = std::log(delta / delta_prev) / (double)(it - it_prev);   // < 0
      const double to_go = std::log(st[ST_STOP] / delta) / per_it;                    // > 0
      if (to_go < 1e9) need = std::max<int64_t>(1, (int64_t)std::ceil(1.25 * to_go));
    }
    it_prev = it;
    delta_prev = delta;
  }
  CgEnd e;
  e.it = it;
  e.extra_products = extra_products;
  e.converged = done && !broke && !stalled;
  e.broke = broke;
  e.stalled = stalled;
  e.delta0 = delta0;
  e.delta = delta;
  e.t_setup = t_setup;
  e.t_cg = ms_since(t1);
  e.t_matvec = tm.total_ms;
  e.n_timed = tm.count;
  LSSVM_TRY(end_cg<T>(g, w, e, status, info, t0, s));
  if (stalled)   // the iterate of the smallest recomputed residual, whose r^T r was reported
    LSSVM_HIP(hipMemcpyAsync(w.x, w.xbest, NP * sizeof(double), hipMemcpyDeviceToDevice, s));

  // ---- a6: alpha_m and b
  LSSVM_HIP(launch_bias<T>(w.x, w.q64, g.N, y, w.scal, 1.0 / C, alpha_out, s));
  LSSVM_HIP(launch_read_back(w.scal + S_B, 1, g_ctx->p, s));
  LSSVM_HIP(hipStreamSynchronize(s));
  *b_out = g_ctx->p[0];
  end_report(g, e, info, t0);
  if (info && info->compute_true_residual) {
    if (delta0 > 0.0) {
      if (passes) LSSVM_TRY(lin.product(w.x, false));
      else LSSVM_TRY(matvec_partials<T>(g, w, kp, kernel, w.x, s));
    }
    LSSVM_TRY(true_residual<T>(g, w, product_of(w.x), NP, delta0, info, s));
  }
  return e.status;
}

// Workspace of lssvm_cg_step: the scalar area and two block-partial arrays.
constexpr int64_t kMaxStepLen = int64_t(1) << 34;
struct StepWs {
  double *scal, *bp0, *bp1;
  size_t bytes;
};
StepWs carve_step(int64_t N, void* base) {
  Carver c(base);
  StepWs w{};
  const int64_t nb = vec_blocks(N);
  w.scal = c.take<double>(S_COUNT);
  w.bp0 = c.take<double>(nb + 1);
  w.bp1 = c.take<double>(nb + 1);
  w.bytes = c.off;
  return w;
}

bool overlaps(const void* a, const void* b, int64_t bytes) {
  const char* pa = static_cast<const char*>(a);
  const char* pb = static_cast<const char*>(b);
  return pa < pb + bytes && pb < pa + bytes;
}

template <typename T>
int matvec_impl(const T* X, int64_t n, int64_t d, int32_t kernel, const lssvm_params& kp,
                double C, const T* p, T* out, void* workspace, size_t ws_bytes, hipStream_t s) {
  const Geometry g = geometry<T>(n, d);
  TrainWs<T> w = carve_train<T>(g, nullptr);
  LSSVM_TRY(check_workspace(workspace, ws_bytes, w.bytes));
  w = carve_train<T>(g, workspace);
  LSSVM_HIP(g_ctx->ensure());
  if (linear_passes(g, kernel)) {   // out stays untouched if X is not finite: one wait, at the end
    const LinearPasses<T> lin(g, w, X, C, s);
    LSSVM_HIP(launch_setup_clear(0, LSSVM_TILE_GROUP, nullptr, w.flags, w.scal, nullptr, 0,
                                 nullptr, s));
    LSSVM_HIP(launch_lin_q<T>(X, g.n, g.d, w.q64, w.scal, w.flags, s));
    LSSVM_HIP(launch_pad_to_f64<T>(p, g.N, w.dir, g.N, nullptr, nullptr, s));
    LSSVM_HIP(lin.weights(lin.vec(w.dir, false)));
    LSSVM_HIP(launch_lin_out<T>(X, g.N, g.d, w.lin_w, lin.rank_one(w.dir, nullptr), out, w.flags,
                                s));
    LSSVM_HIP(read_flags(w.flags, s));
    LSSVM_HIP(hipStreamSynchronize(s));
    if (g_ctx->flags[F_NONFINITE]) return fail(LSSVM_ENONFINITE, "X holds a NaN or an infinity");
    return LSSVM_OK;
  }
  LSSVM_TRY(setup_points<T>(g, w, X, kernel, kp, s));
  LSSVM_HIP(launch_pad_to_f64<T>(p, g.N, w.dir, g.NP, w.scal, w.flags, s));
  for (bool again = false;; again = true) {   // one wait, at the end
    TileArgs<T> a = sym_args<T>(g, w, kp, kernel, w.dir);
    if (!again) a.stop = w.scal + S_STATUS + ST_DONE;
    LSSVM_HIP(launch_product<T>(g, a, kernel, w.gpart, s));
    LSSVM_HIP(launch_mv_out<T>(rank_one(g, w, kernel, C, w.dir), g.NP, g.N, out, s));
    LSSVM_HIP(read_flags(w.flags, s));
    LSSVM_HIP(hipStreamSynchronize(s));
    if (g_ctx->flags[F_NONFINITE]) return fail(LSSVM_ENONFINITE, "X holds a NaN or an infinity");
    if (!g_ctx->flags[F_RANGE]) return LSSVM_OK;
    LSSVM_TRY(rescale_points<T>(g, w, X, kernel, kp, s));   // the product has waited for this
  }
}

// Whether a prediction takes k_predict_few, which reads the model once but gives
// every point its own epilogue in the registers of one (fp64) or two workgroups
// per CU: up to 64 points nearly always. From 65 on its instance holds 128 points
// and a round of workgroups covers 8192 (fp64) or 16384 model points, about 40 us
// each; the tiles pay for the layout instead, which many features make dear. Call
// times on the tiles and so, 128 points: cubic fp64 8192 x 30 46 and 41 us, 12000 x
// 30 48 and 54, 50000 x 30 62 and 114, 16384 x 1000 216 and 153; cubic fp32 16384 x
// 30 47 and 41, 50000 x 30 57 and 68; RBF fp64 24500 x 30 67 and 62, 50000 x 30 84
// and 102; RBF fp32 50000 x 30 79 and 68. 64 points of fp64 RBF: 100000 x 30 105
// and 102, 200000 x 30 150 and 171.
inline bool few_points(int32_t kernel, bool fp64, int64_t n, int64_t d, int64_t n_test) {
  const int64_t round = fp64 ? 8192 : 16384;
  if (kernel == LSSVM_LINEAR || n_test > kFewTests) return false;
  if (n_test > 64) {
    if (kernel == LSSVM_POLY) return n <= round * (d < 512 ? 1 : d < 1000 ? 2 : 3);
    return d >= 1000 || n <= 3 * round;
  }
  return !(n_test > 32 && kernel == LSSVM_RBF && fp64 && d < 128) || n <= 12 * round;
}

template <typename T>
int predict_impl(const T* Xtr, const T* alpha, double b, int64_t n, int64_t d, int32_t kernel,
                 const lssvm_params& kp, const T* Xte, int64_t n_test, void* workspace,
                 size_t ws_bytes, T* scores, int32_t* labels, hipStream_t s) {
  const Geometry g = geometry<T>(n, d);
  PredictWs<T> w = carve_predict<T>(g, n_test, nullptr);
  LSSVM_TRY(check_workspace(workspace, ws_bytes, w.bytes));
  w = carve_predict<T>(g, n_test, workspace);
  LSSVM_HIP(g_ctx->ensure());
  if (few_points(kernel, sizeof(T) == 8, n, d, n_test)) {
    PredictFew<T> a{};
    a.Xtr = Xtr;
    a.Xte = Xte;
    a.alpha = alpha;
    a.n = n;
    a.n_test = n_test;
    a.d = d;
    a.gamma = kp.gamma;
    a.coef0 = kp.coef0;
    a.rbf_scale = rbf_scale<T>(kp.gamma);
    a.degree = kp.degree;
    a.part = w.few_part;
    a.bad = w.few_bad;
    LSSVM_HIP(launch_predict_few<T>(a, kernel, b, scores, labels, w.flags, s));
    LSSVM_HIP(read_flags(w.flags, s));
    LSSVM_HIP(hipStreamSynchronize(s));
    if (g_ctx->flags[F_NONFINITE])
      return fail(LSSVM_ENONFINITE, "X_train or X_test holds a NaN or an infinity");
    return LSSVM_OK;
  }
  LSSVM_HIP(hipMemsetAsync(w.flags, 0, F_COUNT * sizeof(int), s));
  if (kernel == LSSVM_LINEAR) {  // Eq. (15): w = sum_i alpha_i x_i, f(x) = <w, x> + b
    LSSVM_HIP(launch_linear_predict<T>(Xtr, alpha, n, d, Xte, n_test, b, w.lin_part, w.lin_w,
                                       w.lin_f, scores, labels, w.flags, s));
    LSSVM_HIP(read_flags(w.flags, s));
    LSSVM_HIP(hipStreamSynchronize(s));
    if (g_ctx->flags[F_NONFINITE])
      return fail(LSSVM_ENONFINITE, "X_train or X_test holds a NaN or an infinity");
    return LSSVM_OK;
  }
  LSSVM_HIP(launch_layout<T>(Xtr, n, d, w.Xtr, g.ld, g.d_pad, kStoredUp<T>, 1, w.flags, s));
  LSSVM_HIP(launch_layout<T>(Xte, n_test, d, w.Xte, w.ld_te, g.d_pad, kStoredUp<T>, 1, w.flags, s));
  auto norms = [&](int up_tr, int up_te) {   // only the radial kernel reads them
    if (kernel != LSSVM_RBF) return hipSuccess;
    const hipError_t e = launch_norms_q<T>(w.Xtr, g.ld, g.d_pad, -1, 0, up_tr, kernel, kp.gamma,
                                           kp.coef0, kp.degree, w.ntr, nullptr, nullptr, s);
    if (e != hipSuccess) return e;
    return launch_norms_q<T>(w.Xte, w.ld_te, g.d_pad, -1, 0, up_te, kernel, kp.gamma, kp.coef0,
                             kp.degree, w.nte, nullptr, nullptr, s);
  };
  int up_tr = kStoredUp<T>, up_te = kStoredUp<T>;
  LSSVM_HIP(norms(up_tr, up_te));
  LSSVM_HIP(launch_pad_vec<T>(alpha, n, w.alpha, g.ld, w.flags, w.wait, s));
  TileArgs<T> a{};
  a.A = w.Xte;
  a.B = w.Xtr;
  a.nkb = g.d_pad / TileShape<T>::SB;
  a.nA = w.nte;
  a.nB = w.ntr;
  a.wB = w.alpha;
  a.gscale = (T)std::ldexp(1.0, -up_tr - up_te);
  a.gamma = (T)kp.gamma;
  a.coef0 = (T)kp.coef0;
  a.gamma64 = kp.gamma;
  a.coef64 = kp.coef0;
  a.rbf_scale = rbf_scale<T>(kp.gamma);
  a.degree = kp.degree;
  a.nTc = w.nTc;
  a.ksplit = 1;
  a.part = w.part;
  a.part_ld = w.ld_te;
  a.stop = w.wait;
  for (;;) {
    LSSVM_HIP(launch_tiles_gen<T>(a, kernel, w.nTr, s));
    LSSVM_HIP(launch_predict_finish<T>(w.part, w.nTc, w.ld_te, n_test, b, scores, labels, w.flags,
                                       s));
    LSSVM_HIP(read_flags(w.flags, s));
    LSSVM_HIP(hipStreamSynchronize(s));
    if (g_ctx->flags[F_NONFINITE])
      return fail(LSSVM_ENONFINITE, "X_train or X_test holds a NaN or an infinity");
    if (!g_ctx->flags[F_RANGE]) return LSSVM_OK;
    // out of the usual range on either side: the scores have waited for this
    LSSVM_TRY(relayout(Xtr, n, d, w.Xtr, g.ld, g.d_pad, w.flags, &up_tr, s));
    LSSVM_TRY(relayout(Xte, n_test, d, w.Xte, w.ld_te, g.d_pad, w.flags, &up_te, s));
    LSSVM_HIP(norms(up_tr, up_te));
    a.gscale = (T)std::ldexp(1.0, -up_tr - up_te);
    a.stop = nullptr;
  }
}

template <typename T>
size_t train_bytes(int64_t n, int64_t d) {
  return carve_train<T>(geometry<T>(n, d), nullptr).bytes;
}

template <typename T>
size_t predict_bytes(int64_t n, int64_t n_test, int64_t d) {
  return carve_predict<T>(geometry<T>(n, d), n_test, nullptr).bytes;
}

lssvm_params params_or_default(const lssvm_params* kp) {
  lssvm_params p{1.0, 0.0, 1};
  if (kp) p = *kp;
  return p;
}

}  // namespace
}  // namespace lssvm

using namespace lssvm;

extern "C" {

size_t lssvm_cg_step_workspace_bytes(int64_t N) {
  if (N < 1 || N > kMaxStepLen) return 0;
  return carve_step(N, nullptr).bytes;
}

int lssvm_cg_step(int64_t N, double* x, double* r, double* d, const double* q, double* scalars,
                  void* workspace, size_t workspace_bytes, void* stream) {
  try {
    g_last_error.clear();
    if (!x || !r || !d || !q || !scalars) return fail(LSSVM_EINVAL, "NULL array argument");
    if (N < 1 || N > kMaxStepLen)
      return fail(LSSVM_EINVAL, "N must be in [1, 2^34] (got %lld)", (long long)N);
    const void* v[4] = {x, r, d, q};
    for (int i = 0; i < 4; ++i)
      for (int j = i + 1; j < 4; ++j)
        if (overlaps(v[i], v[j], N * (int64_t)sizeof(double)))
          return fail(LSSVM_EINVAL, "x, r, d and q must not overlap");
    StepWs w = carve_step(N, workspace);
    LSSVM_TRY(check_workspace(workspace, workspace_bytes, w.bytes));
    LSSVM_HIP(launch_cg_step(N, x, r, d, q, scalars, w.scal, w.bp0, w.bp1,
                             static_cast<hipStream_t>(stream)));
    return LSSVM_OK;
  } catch (...) {
    return fail(LSSVM_EHIP, "internal error");
  }
}

int lssvm_cg_step_noalloc(int64_t N, double* x, double* r, double* d, const double* q,
                          double* scalars, void* stream) {
  try {
    g_last_error.clear();
    if (!x || !r || !d || !q || !scalars) return fail(LSSVM_EINVAL, "NULL array argument");
    if (N < 1 || N > kMaxStepLen)
      return fail(LSSVM_EINVAL, "N must be in [1, 2^34] (got %lld)", (long long)N);
    const void* v[4] = {x, r, d, q};
    for (int i = 0; i < 4; ++i)
      for (int j = i + 1; j < 4; ++j)
        if (overlaps(v[i], v[j], N * (int64_t)sizeof(double)))
          return fail(LSSVM_EINVAL, "x, r, d and q must not overlap");
    double* base = nullptr;
    int64_t capacity = 0;
    LSSVM_HIP(static_scratch(&base, &capacity));
    const size_t need = carve_step(N, nullptr).bytes;
    if (need > (size_t)capacity * sizeof(double))
      return fail(LSSVM_EINVAL, "N = %lld needs %zu bytes of scratch, above the %lld held",
                  (long long)N, need, (long long)(capacity * (int64_t)sizeof(double)));
    StepWs w = carve_step(N, base);
    LSSVM_HIP(launch_cg_step(N, x, r, d, q, scalars, w.scal, w.bp0, w.bp1,
                             static_cast<hipStream_t>(stream)));
    return LSSVM_OK;
  } catch (...) {
    return fail(LSSVM_EHIP, "internal error");
  }
}

int64_t lssvm_host_contexts(void) { return g_pool_size.load(); }

size_t lssvm_workspace_bytes(int64_t n, int64_t d, int32_t dtype) {
  if (n < 1 || d < 1 || n > kMaxPoints || d > kMaxFeatures || !valid_dtype(dtype)) return 0;
  return dtype == LSSVM_F64 ? train_bytes<double>(n, d) : train_bytes<float>(n, d);
}

size_t lssvm_predict_workspace_bytes(int64_t n, int64_t n_test, int64_t d, int32_t dtype) {
  if (n < 1 || n_test < 1 || d < 1 || n > kMaxPoints || n_test > kMaxPoints ||
      d > kMaxFeatures || !valid_dtype(dtype))
    return 0;
  return dtype == LSSVM_F64 ? predict_bytes<double>(n, n_test, d)
                            : predict_bytes<float>(n, n_test, d);
}

int32_t lssvm_tile_size(int32_t dtype) {
  if (dtype == LSSVM_F64) return TileShape<double>::T;
  if (dtype == LSSVM_F32) return TileShape<float>::T;
  return 0;
}

int lssvm_tile_plan(int64_t n, int64_t d, int32_t dtype, int32_t kernel, int64_t* plan) {
  clear_error();
  if (n < 2 || d < 1 || n > kMaxPoints || d > kMaxFeatures)
    return fail(LSSVM_EINVAL, "tile_plan: need 2 <= n <= 2^22 and 1 <= d <= 2^21");
  if (kernel != LSSVM_LINEAR && kernel != LSSVM_POLY && kernel != LSSVM_RBF)
    return fail(LSSVM_EINVAL, "tile_plan: unknown kernel");
  if (dtype != LSSVM_F64 && dtype != LSSVM_F32) return fail(LSSVM_EINVAL, "tile_plan: unknown dtype");
  if (!plan) return fail(LSSVM_EINVAL, "tile_plan: null plan");
  const Geometry g = dtype == LSSVM_F64 ? geometry<double>(n, d) : geometry<float>(n, d);
  const bool lin = kernel == LSSVM_LINEAR;
  plan[0] = linear_passes(g, kernel) ? 0 : product_split(g, kernel);
  plan[1] = lin ? 0 : g.part_q;
  plan[2] = plan[1] == 0 ? plan[0] : g.part_split;
  return LSSVM_OK;
}

const char* lssvm_last_error(void) { return g_last_error.c_str(); }

int lssvm_train(const void* X, const void* y, int64_t n, int64_t d, int32_t dtype,
                int32_t kernel, const lssvm_params* kp, double C, double eps, int64_t max_iter,
                void* workspace, size_t workspace_bytes, void* alpha_out, double* b_out,
                lssvm_info* info, void* stream) {
  try {
    g_last_error.clear();
    if (!X || !y || !alpha_out || !b_out) return fail(LSSVM_EINVAL, "NULL array argument");
    if (!valid_dtype(dtype)) return fail(LSSVM_EINVAL, "unknown dtype %d", (int)dtype);
    LSSVM_TRY(check_sizes(n, d, 1));
    LSSVM_TRY(check_kernel_params(kernel, kp));
    if (!(C > 0.0) || !std::isfinite(C)) return fail(LSSVM_EINVAL, "C must be finite and > 0");
    if (!(eps > 0.0 && eps < 1.0)) return fail(LSSVM_EINVAL, "eps must lie in (0, 1)");
    if (max_iter < 0) return fail(LSSVM_EINVAL, "max_iter must be >= 0");
    if (info && info->residual_history == nullptr && info->history_capacity != 0)
      return fail(LSSVM_EINVAL, "history_capacity without residual_history");
    if (info && info->matvec_times == nullptr && info->matvec_times_capacity != 0)
      return fail(LSSVM_EINVAL, "matvec_times_capacity without matvec_times");
    const lssvm_params p = params_or_default(kp);
    hipStream_t s = static_cast<hipStream_t>(stream);
    CtxLease lease;
    if (dtype == LSSVM_F64)
      return train_impl<double>(static_cast<const double*>(X), static_cast<const double*>(y), n, d,
                                kernel, p, C, eps, max_iter, workspace, workspace_bytes,
                                static_cast<double*>(alpha_out), b_out, info, s);
    return train_impl<float>(static_cast<const float*>(X), static_cast<const float*>(y), n, d,
                             kernel, p, C, eps, max_iter, workspace, workspace_bytes,
                             static_cast<float*>(alpha_out), b_out, info, s);
  } catch (...) {
    return fail(LSSVM_EHIP, "internal error");
  }
}

int lssvm_predict(const void* X_train, const void* alpha, double b, int64_t n, int64_t d,
                  int32_t dtype, int32_t kernel, const lssvm_params* kp, const void* X_test,
                  int64_t n_test, void* workspace, size_t workspace_bytes, void* scores_out,
                  int32_t* labels_out, void* stream) {
  try {
    g_last_error.clear();
    if (!X_train || !alpha || !X_test || !scores_out)
      return fail(LSSVM_EINVAL, "NULL array argument");
    if (!valid_dtype(dtype)) return fail(LSSVM_EINVAL, "unknown dtype %d", (int)dtype);
    LSSVM_TRY(check_sizes(n, d, 1));
    if (n_test < 1 || n_test > kMaxPoints)
      return fail(LSSVM_EINVAL, "n_test must be in [1, 2^22] (got %lld)", (long long)n_test);
    LSSVM_TRY(check_kernel_params(kernel, kp));
    if (!std::isfinite(b)) return fail(LSSVM_EINVAL, "b must be finite");
    const lssvm_params p = params_or_default(kp);
    hipStream_t s = static_cast<hipStream_t>(stream);
    CtxLease lease;
    if (dtype == LSSVM_F64)
      return predict_impl<double>(static_cast<const double*>(X_train),
                                  static_cast<const double*>(alpha), b, n, d, kernel, p,
                                  static_cast<const double*>(X_test), n_test, workspace,
                                  workspace_bytes, static_cast<double*>(scores_out), labels_out,
                                  s);
    return predict_impl<float>(static_cast<const float*>(X_train),
                               static_cast<const float*>(alpha), b, n, d, kernel, p,
                               static_cast<const float*>(X_test), n_test, workspace,
                               workspace_bytes, static_cast<float*>(scores_out), labels_out, s);
  } catch (...) {
    return fail(LSSVM_EHIP, "internal error");
  }
}

int lssvm_matvec(const void* X, int64_t n, int64_t d, int32_t dtype, int32_t kernel,
                 const lssvm_params* kp, double C, const void* p, void* out, void* workspace,
                 size_t workspace_bytes, void* stream) {
  try {
    g_last_error.clear();
    if (!X || !p || !out) return fail(LSSVM_EINVAL, "NULL array argument");
    if (!valid_dtype(dtype)) return fail(LSSVM_EINVAL, "unknown dtype %d", (int)dtype);
    LSSVM_TRY(check_sizes(n, d, 2));
    LSSVM_TRY(check_kernel_params(kernel, kp));
    if (!(C > 0.0) || !std::isfinite(C)) return fail(LSSVM_EINVAL, "C must be finite and > 0");
    const lssvm_params pr = params_or_default(kp);
    hipStream_t s = static_cast<hipStream_t>(stream);
    CtxLease lease;
    if (dtype == LSSVM_F64)
      return matvec_impl<double>(static_cast<const double*>(X), n, d, kernel, pr, C,
                                 static_cast<const double*>(p), static_cast<double*>(out),
                                 workspace, workspace_bytes, s);
    return matvec_impl<float>(static_cast<const float*>(X), n, d, kernel, pr, C,
                              static_cast<const float*>(p), static_cast<float*>(out), workspace,
                              workspace_bytes, s);
  } catch (...) {
    return fail(LSSVM_EHIP, "internal error");
  }
}

}  // extern "C"
