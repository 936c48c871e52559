// Internal interface between the host runtime (api.cpp) and the gfx950
// kernels (kernels.hip). Not part of the public C ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

#include "tile_args.h"

namespace lssvm {

// Symmetric tiles are visited in GROUP x GROUP super-tiles of the upper
// triangle, and each of the 8 XCDs takes a contiguous run of that order, so
// the workgroups resident on one XCD share few point panels in its L2.
// 0 = plain column-by-column triangle order, no remap.
#ifndef LSSVM_TILE_GROUP
#define LSSVM_TILE_GROUP 8
#endif

// Slots of the small fp64 scalar area in the workspace.
enum Scalar : int {
  S_KMM = 0,     // k(x_m, x_m)
  S_DHIST = 1,   // r^T r of the current iterate, double-buffered: [1], [2]
  S_DELTA0 = 3,  // r0^T r0
  S_B = 4,       // bias
  S_ALPHA = 5,   // CG step length of the last update
  S_GAMMA = 6,   // curvature d^T Q~ d of the last update
  S_TRUE = 7,    // ||rhs - Q~ x||^2 (final report)
  S_STATUS = 8,  // 8 doubles read by the host after each batch of iterations:
                 // [0] r^T r of the last iteration run (on a stall: that of the
                 // best recomputed residual), [1] its curvature, [2] its step
                 // length, [3] its number, [4] done (converged, broken down or
                 // stalled), [5] breakdown, [6] stop threshold eps^2 r0^T r0,
                 // [7] stalled
  S_BEST = 16,   // smallest true r^T r so far (start, residual recomputations),
                 // double-buffered by recomputation: [16], [17]
  S_PHI = 18,    // smallest CG energy -(rhs + r)^T x / 2 so far, likewise: [18], [19]
  // Fixed-point row sums of the symmetric products (tiles.h): [20] max |p_j| of
  // the vector the next product multiplies (raised with an integer atomic max
  // on its bits by the kernel that writes the vector, cleared by the kernel
  // that reads the product), [21] max ||x_i||^2, [22] the scale 2^s the last
  // product used
  S_PMAX = 20,
  S_NMAX = 21,
  S_FIXSC = 22,
  S_INFLAGS = 23,   // the input flags as read after the right-hand side: 1 non-finite
                    // X, 2 a label other than +-1, 4 F_RANGE (one read-back with S_DELTA0)
  S_TIMES = 24,     // k_lin_train: wall clock ticks of its setup, and of the rest
  S_COUNT = 26
};
enum StatusField : int { ST_DELTA = 0, ST_CURV = 1, ST_STEP = 2, ST_ITER = 3, ST_DONE = 4,
                         ST_BREAK = 5, ST_STOP = 6, ST_STALL = 7, ST_COUNT = 8 };

// The CG vector kernels run at most this many blocks of 256 threads (4 per
// CU), each striding over the vector, so every block can re-sum the previous
// kernel's block partials cheaply at any vector length.
constexpr int64_t kVecBlocks = 1024;
inline int64_t vec_blocks(int64_t len) {
  const int64_t b = (len + 255) / 256;
  return b < kVecBlocks ? (b > 0 ? b : 1) : kVecBlocks;
}

// The training's CG vector kernels (the readers of a product included: each
// row's sum is two words) run one block per 256 rows of the padded vectors,
// at most kVecBlocks, striding beyond that.
inline int64_t cg_blocks(int64_t NP) { return vec_blocks(NP); }

// Flags raised by kernels (int32 each).
// F_PRODUCT: a symmetric product had a row sum that is not finite (its
// entries then come out as NaN, so CG reports a breakdown).
// F_RANGE: an fp32 point holds a value that the usual stored scale does not serve
// (kSplitMin, kSplitMax), and the points are not yet laid out to suit (products and
// scores wait for that: TileArgs::stop).
enum Flag : int { F_NONFINITE = 0, F_BADLABEL = 1, F_PRODUCT = 2, F_RANGE = 3, F_COUNT = 4 };


// One symmetric product as its readers see it: (K p)_i in the fixed-point
// accumulators of the tiles, and the rank-one and diagonal terms of Q~ p that
// the tiles leave out (Eq. (13)): (Q~ p)_i = (K p)_i + (Q_mm - q_i) S - T +
// p_i / C for i < N, with S = sum_j p_j, T = sum_j q_j p_j (summed from the
// diagonal tiles' per-panel partials in a fixed order) and
// Q_mm = k(x_m, x_m) + 1/C. A reader clears the accumulators it reads.
struct RankOne {
  const double* pq;    // 2 nT panel partials: S_I, then T_I
  int64_t nT;
  int64_t* acc;        // fixed-point row sums (two words per row)
  const double* q64;   // q_i, zero beyond N
  const double* p;     // the vector multiplied, zero beyond N
  double* scal;        // k(x_m, x_m) at S_KMM, the product's scale at S_FIXSC
  const int* flags;    // F_PRODUCT
  double invC;
  const double* kp;    // (K p)_i itself (linear products), or null: from acc
};

// The vector a linear product multiplies: p, or, with dir_out, the new CG
// direction r + beta p, which is written to dir_out. beta and the status come
// from the last update's block partials (bp, nb) as in k_cg_direction, whose
// iteration `iter` (r^T r before it in S_DHIST + par) this ends.
struct LinVec {
  const double* p;
  const double* r;
  double* dir_out;
  const double* bp;
  int64_t nb;
  double* scal;
  int par, stop;      // stop: return at once when CG has stopped
  int64_t iter;
  double* hist;
  int64_t hist_cap;
};
// Launch shape of w = X^T p: column blocks, row chunks, rows per chunk.
struct LinShape {
  int64_t ncb, nch, rows;
};

// One fused CG iteration for small problems (see launch_tiles_cg): the
// product's tiles, then, in the workgroup that finishes last, the vector work
// of k_cg_gather, k_cg_update and k_cg_direction on the whole vectors.
struct FusedCg {
  unsigned* ticket;   // zero before every launch; the last workgroup resets it
  RankOne c;          // c.p = the CG direction
  double *qv, *x, *r, *dir, *scal, *hist;
  int64_t NP, N, iter, hist_cap;
  int par;            // r^T r of the current iterate lives in S_DHIST + par
};
// Largest padded length the fused iteration handles: one workgroup reads every
// row sum and keeps each thread's rows (NP / 256) in registers. Trainings, fused
// and with a launch per vector step: 1900 x 100 fp32 RBF 1.04 and 1.43 ms, 1038 x 66
// fp64 0.94 and 1.09, 2040 x 50 1.21 and 1.28. (At 4096 points the release and
// ticket of each of the workgroups made the launch ~50 us longer than the
// product, more than the launches cost.)
constexpr int64_t kFusedMaxNP = 2048;
// ... of the linear kernel, whose larger problems are passes over the points.
constexpr int64_t kFusedMaxLinear = 1024;

// The symmetric tiles' visit order (GROUP x GROUP super-tiles), packed
// (I << 16) | J, nT (nT + 1) / 2 entries.
// The first kernel of a training: zeroes the flags (F_COUNT ints), the
// scalars (S_COUNT doubles), the row-sum words (nacc int64) and the fused
// iteration's ticket (if given), and writes the tile visit order (order may
// be null: then nothing but the zeroing).
hipError_t launch_setup_clear(int64_t nT, int64_t group, uint32_t* order,
                              int* flags, double* scal, int64_t* acc, int64_t nacc,
                              unsigned* ticket, hipStream_t s);

// fp32 values are stored multiplied by 2^up; check: raise F_RANGE.
template <typename T> constexpr int kStoredUp = sizeof(T) == 4 ? 16 : 0;
template <typename T>
hipError_t launch_layout(const T* X, int64_t n, int64_t d, store_t<T>* Xt, int64_t ld, int64_t d_pad,
                         int up, int check, int* flags, hipStream_t s);
// Raises *out (an int32 set to 0 before) to the bits of the largest |X[k]| of
// `count` values.
hipError_t launch_abs_max(const float* X, int64_t count, int* out, hipStream_t s);
template <typename T>
hipError_t launch_norms_q(const store_t<T>* Xt, int64_t ld, int64_t d_pad, int64_t m, int64_t N,
                          int up, int kernel, double gamma, double coef0, int degree, T* norms,
                          double* q64, double* scal, hipStream_t s);
template <typename T>
// Symmetric tile launch of nwg workgroups doing `part` (a TilePart; a fixup
// launch has one workgroup per tile).
hipError_t launch_tiles_sym(const TileArgs<T>& a, int kernel, int part, int64_t nwg,
                            hipStream_t s);
template <typename T>
hipError_t launch_tiles_gen(const TileArgs<T>& a, int kernel, int64_t nTr, hipStream_t s);
// A whole CG iteration for small problems (NP <= kFusedMaxNP) in one launch of
// whole tiles, or in the fixup launch of split ones: the symmetric tiles of q =
// Q~ d, then the workgroup that finishes last (an atomic ticket after a
// device-scope release fence) adds the rank-one terms and does the update and the new direction, with the same
// status, stop test and breakdown handling as the separate kernels. Nothing
// waits on another workgroup.
template <typename T>
hipError_t launch_tiles_cg(const TileArgs<T>& a, int kernel, int part, int64_t nwg,
                           const FusedCg& f, hipStream_t s);
// rhs = ybar - y_m 1, x = xbest = 0, r = dir = rhs, the block partials of
// r^T r; raises scal[S_PMAX] to max |dir| (the first product multiplies it).
template <typename T>
hipError_t launch_rhs_init(const T* y, int64_t N, int64_t NP, double* rhs, double* x,
                           double* xbest, double* r, double* dir, double* bpart, int* flags,
                           double* scal, hipStream_t s);
// CG kernels: once the status says done, every later kernel of the queue
// returns at once, so the host may enqueue iterations ahead of the test.
hipError_t launch_finish_delta0(const double* bpart, int64_t nb, double* scal, double eps2,
                                const int* flags, hipStream_t s);
// q = Q~ dir (c.p = dir) and the block partials of dir^T q.
hipError_t launch_cg_gather(const RankOne& c, int64_t NP, int64_t N, double* qv, double* bpart,
                            hipStream_t s);
hipError_t launch_cg_update(int x_only, const double* bp_in, int64_t nb, double* scal, int par,
                            const double* dir, const double* qv, double* x, double* r,
                            double* bp_out, int64_t NP, hipStream_t s);
// r = rhs - Q~ x (c.p = x), the block partials of r^T r and those of
// (rhs + r)^T x (minus twice the CG energy of x).
hipError_t launch_cg_residual(const RankOne& c, int64_t NP, int64_t N, const double* rhs, double* r,
                              double* bp_out, double* bp_phi, hipStream_t s);
// Warm start: delta = r0^T r0 from the block partials, dir = r0, the start as
// the best iterate so far (its residual and energy), done if already below
// the stop threshold.
hipError_t launch_warm_start(const double* bp_in, const double* bp_phi, int64_t nb, double* scal,
                             const double* r, double* dir, const double* x, double* xbest,
                             int64_t NP, hipStream_t s);
// One CG iteration on caller vectors of length N given q = A d: the scalars
// (device, 4 doubles) carry r^T r in and r^T r, d^T q, step, beta out.
hipError_t launch_cg_step(int64_t N, double* x, double* r, double* d, const double* q,
                          double* scalars, double* scal, double* bp0, double* bp1,
                          hipStream_t s);
// beta and the new direction; stop on eps. refresh > 0 marks the refresh-th
// residual recomputation: then r is a true residual, bp_phi holds the
// partials of (rhs + r)^T x, and CG stops, stalled, unless the residual or
// the energy sets a new minimum (x is copied to xbest on a new residual
// minimum).
hipError_t launch_cg_direction(const double* bp_in, int64_t nb, double* scal, int par,
                               int64_t iter, const double* r, double* dir, int64_t NP,
                               double* hist, int64_t hist_cap, int64_t refresh, int raise,
                               const double* bp_phi, const double* x, double* xbest,
                               hipStream_t s);
template <typename T>
hipError_t launch_bias(const double* x, const double* q64, int64_t N, const T* y, double* scal,
                       double invC, T* alpha_out, hipStream_t s);
// n = 1: alpha = [0] and b = y_0, alpha written only if the point and its
// label passed the checks (flags set by the layout kernel before it).
template <typename T>
hipError_t launch_single_point(const T* y, T* alpha_out, double* scal, int* flags, hipStream_t s);
// dst = src zero-padded; *wait = 1 if F_RANGE is up, else 0.
template <typename T>
hipError_t launch_pad_vec(const T* src, int64_t len, T* dst, int64_t len_pad, const int* flags,
                          double* wait, hipStream_t s);
template <typename T>
hipError_t launch_mv_out(const RankOne& c, int64_t NP, int64_t N, T* out, hipStream_t s);
// scores = b + the sum of nslots partial slots; nothing is written if the
// input flags report a non-finite point.
template <typename T>
hipError_t launch_predict_finish(const double* part, int64_t nslots, int64_t ld, int64_t n_test,
                                 double b, T* scores, int32_t* labels, const int* flags,
                                 hipStream_t s);
// dst = src zero-padded, in fp64; with scal, also raises scal[S_PMAX] to max |dst|;
// with flags, sets the stop flag (ST_DONE) to 1 if F_RANGE is up.
template <typename T>
hipError_t launch_pad_to_f64(const T* src, int64_t len, double* dst, int64_t len_pad,
                             double* scal, const int* flags, hipStream_t s);
// count <= 64 doubles from the device to pinned host memory, for a host that waits
// for the stream next.
hipError_t launch_read_back(const double* src, int count, double* dst, hipStream_t s);
hipError_t launch_finish_sum(const double* bpart, int64_t nb, double* scal, int slot,
                             hipStream_t s);
hipError_t launch_true_residual(const RankOne& c, int64_t NP, int64_t N, const double* rhs,
                                double* bp_out, hipStream_t s);

// Linear-kernel decision values through w = sum_i alpha_i x_i (Eq. (15)).
// part: lin_max_chunks(n, d) d doubles; w: d doubles; f: n_test
// doubles (the inner products before the bias).
template <typename T>
hipError_t launch_linear_predict(const T* Xtr, const T* alpha, int64_t n, int64_t d, const T* Xte,
                                 int64_t n_test, double b, double* part, double* w, double* f,
                                 T* scores, int32_t* labels, int* flags, hipStream_t s);
// Decision values of at most kFewTests points on a polynomial or RBF model
// (k_predict_few): part holds n_test predict_few_slots(n, n_test) doubles, bad
// as many ints as slots.
constexpr int64_t kFewTests = 128;
template <typename T>
struct PredictFew {
  const T *Xtr, *Xte, *alpha;
  int64_t n, n_test, d;
  int vec;   // set by the launcher
  double gamma, coef0;
  T rbf_scale;
  int degree;
  double* part;
  int* bad;
};
int64_t predict_few_slots(int64_t n, int64_t n_test);
template <typename T>
hipError_t launch_predict_few(PredictFew<T> a, int kernel, double b, T* scores, int32_t* labels,
                              int* flags, hipStream_t s);

// A whole linear training in one workgroup (k_lin_train): what it needs beside
// the points, and where it leaves x, rhs, q and the scalars (the status fields,
// S_KMM, S_DELTA0, S_B, S_INFLAGS, S_TIMES). alpha is written only if the inputs
// passed and CG did not break down.
struct LinTrain {
  double invC, eps2;
  int max_iter, replace_every;   // 64-bit ones cost the loop scalar registers, which spill
                                 // (256 x 64 fp64: 299 us, 277 so)
  double *x, *rhs, *q64, *scal, *hist;
  int64_t hist_cap;
  int* flags;
};
bool lin_train_fits(int64_t n, int64_t d, int64_t elem);
template <typename T>
hipError_t launch_lin_train(const T* X, const T* y, int64_t n, int64_t d, const LinTrain& a,
                            T* alpha_out, hipStream_t s);

// Linear products (two passes over the caller's rows): q_i and k(x_m, x_m) with
// the finite check; w = X^T p (part: lin_max_chunks(N, d) d doubles, pq: S and T
// per chunk); then (K p)_i, (Q~ p)_i with the partials of p^T Q~ p
// (lin_gather_blocks of them), or (Q~ p)_i as T.
int64_t lin_max_chunks(int64_t N, int64_t d);
LinShape lin_shape(int64_t N, int64_t d, int vec);
template <typename T> int lin_vec(const T* X, int64_t d);
template <typename T> int64_t lin_gather_blocks(const T* X, int64_t N, int64_t d);
template <typename T>
hipError_t launch_lin_q(const T* X, int64_t n, int64_t d, double* q64, double* scal, int* flags,
                        hipStream_t s);
template <typename T>
hipError_t launch_lin_w(const T* X, int64_t N, int64_t d, const LinVec& v, const double* q64,
                        double* part, double* w, double* pq, hipStream_t s);
template <typename T>
hipError_t launch_lin_kp(const T* X, int64_t N, int64_t d, const double* w, double* kp,
                         hipStream_t s);
template <typename T>
hipError_t launch_lin_gather(const T* X, int64_t N, int64_t d, const double* w, const RankOne& c,
                             double* qv, double* bp, hipStream_t s);
template <typename T>
hipError_t launch_lin_out(const T* X, int64_t N, int64_t d, const double* w, const RankOne& c,
                          T* out, int* flags, hipStream_t s);

// The device array that lssvm_cg_step_noalloc works in, for the current
// device: its address (resolved once per device) and its size in doubles.
hipError_t static_scratch(double** ptr, int64_t* capacity);

}  // namespace lssvm
