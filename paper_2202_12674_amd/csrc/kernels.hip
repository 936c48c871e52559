// gfx950 (MI355X, CDNA4) kernels of the LS-SVM training hot path.
//
// a1  k_layout        row-major points -> padded feature-blocked layout (Sec. III-A)
// a2  k_norms_q       squared norms, q_i = k(x_i, x_m) and k(x_m, x_m) (Sec. III-C2)
// a3  k_rhs_init      rhs = ybar - y_m 1 (Eq. (14)), CG start vectors
// a4  k_tiles         implicit K p on the matrix cores, one tile of the upper
//                     triangle per workgroup (Sec. III-C1), rows and columns
//                     accumulated from the same tile; k_cg_gather adds the
//                     rank-one and diagonal terms that make it Q~ p (Eqs. (13), (16))
// a5  k_cg_*          CG vector updates with fixed-order fp64 reductions (Sec. III-B)
// a6  k_bias          alpha_m and b (Eqs. (11), (15))
// a7  k_tiles<gen>    decision values sum_j alpha_j k(x_j, x) + b (Eq. (10));
//     k_predict_few   the same for up to 128 points, from the caller's rows
// Linear kernel: k_lin_w, k_lin_rows (products and decision values through w =
// X^T p), k_lin_train (a whole small training in one workgroup).
//
// Every reduction sums in a fixed order (no floating-point atomics), so the
// results are bitwise reproducible run to run.
#include "lssvm_internal.h"
#include "tiles.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <mutex>
#include <type_traits>

namespace lssvm {

namespace {

constexpr int NT = 256;  // threads per block of the vector kernels

// fp64 kernel value from a dot product and a directly summed squared distance.
template <int KER>
__device__ inline double kernel_value64(double dot, double dist, double gamma, double coef0,
                                        int degree) {
  if constexpr (KER == KLIN) {
    return dot;
  } else if constexpr (KER == KPOLY) {
    const double base = gamma * dot + coef0;
    double r = base;
    for (int e = 1; e < degree; ++e) r *= base;
    return r;
  } else {
    return exp(-gamma * dist);
  }
}

// A commutative operation over the 64 lanes of a wave, every lane receiving
// the result: the 8-lane half rows (DPP: half mirror, then the two quad
// exchanges), the 16-lane rows (DPP rotate by 8), then row pairs and wave
// halves (permlane swaps). Each step combines a lane's value with its
// partner's, and both partners combine the same two values, so all lanes end
// with the same bits. Cross-lane moves in registers: no LDS round trip per
// step, as a shuffle would take.
template <typename Op>
__device__ inline double wave_reduce(double v, Op op) {
  v = op(v, dpp_move<kDppRowHalfMirror>(v));
  v = op(v, dpp_move<kDppQuadXor1>(v));
  v = op(v, dpp_move<kDppQuadXor2>(v));
  v = op(v, dpp_move<kDppRowRor8>(v));
  {
    const uint64_t u = as_u64(v);
    const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)u, (uint32_t)u, false, false);
    const auto hi =
        __builtin_amdgcn_permlane16_swap((uint32_t)(u >> 32), (uint32_t)(u >> 32), false, false);
    v = op(as_f64(lo[0], hi[0]), as_f64(lo[1], hi[1]));   // rows 2k and 2k + 1
  }
  {
    const uint64_t u = as_u64(v);
    const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)u, (uint32_t)u, false, false);
    const auto hi =
        __builtin_amdgcn_permlane32_swap((uint32_t)(u >> 32), (uint32_t)(u >> 32), false, false);
    v = op(as_f64(lo[0], hi[0]), as_f64(lo[1], hi[1]));   // the two halves
  }
  return v;
}
struct AddOp {
  __device__ double operator()(double a, double b) const { return a + b; }
};
struct MaxOp {
  __device__ double operator()(double a, double b) const { return fmax(a, b); }
};
__device__ inline double wave_sum(double v) { return wave_reduce(v, AddOp{}); }

__device__ inline double sum_lanes(double s, int lanes) {   // over 1, 2, 4, 8 or 16 lanes
  if (lanes >= 2) s += dpp_move<kDppQuadXor1>(s);
  if (lanes >= 4) s += dpp_move<kDppQuadXor2>(s);
  if (lanes >= 8) s += dpp_move<kDppRowHalfMirror>(s);
  if (lanes >= 16) s += dpp_move<kDppRowRor8>(s);
  return s;
}

// Block-wide sum of one double per thread; every thread gets the result.
// Fixed reduction order, so every block that sums the same values agrees.
__device__ inline double block_sum(double v, double* sh) {
  v = wave_sum(v);
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  __syncthreads();
  if (l == 0) sh[w] = v;
  __syncthreads();
  double s = 0.0;
  for (int i = 0; i < (int)(blockDim.x >> 6); ++i) s += sh[i];
  return s;
}

// Sum of the nb per-block partials written by the previous kernel.
__device__ inline double sum_partials(const double* bp, int64_t nb, double* sh) {
  double v = 0.0;
  for (int64_t i = threadIdx.x; i < nb; i += blockDim.x) v += bp[i];
  return block_sum(v, sh);
}

// Block-wide S, T and Q_mm of the rank-one terms (every block sums the
// panel partials in the same order, so all blocks agree).
struct RankOneSums {
  double S, Tq, qmm;
};
__device__ inline RankOneSums rank_one_sums(const RankOne& c, double* sh) {
  RankOneSums r;
  r.S = sum_partials(c.pq, c.nT, sh);
  r.Tq = sum_partials(c.pq + c.nT, c.nT, sh);
  r.qmm = c.scal[S_KMM] + c.invC;
  return r;
}
// (Q~ p)_i from the tile sum (K p)_i, for i < N.
__device__ inline double qtilde_row(const RankOne& c, const RankOneSums& r, int64_t i, double kp) {
  return kp + (r.qmm - c.q64[i]) * r.S - r.Tq + c.p[i] * c.invC;
}

// Block-wide maximum of one non-negative double per thread; every thread
// gets it.
__device__ inline double block_max(double v, double* sh) {
  v = wave_reduce(v, MaxOp{});
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  __syncthreads();
  if (l == 0) sh[w] = v;
  __syncthreads();
  double m = 0.0;
  for (int i = 0; i < (int)(blockDim.x >> 6); ++i) m = fmax(m, sh[i]);
  return m;
}

// The stop flag, as one thread of the block reads it: in a launch that may raise
// the flag itself, waves that each read it could disagree, and those that stay
// would sum over a partial that the others never wrote.
__device__ inline bool block_stopped(const double* scal) {
  __shared__ int stopped;
  if (threadIdx.x == 0) stopped = scal[S_STATUS + ST_DONE] != 0.0;
  __syncthreads();
  return stopped != 0;
}

// Raise scal[S_PMAX], the bound on |p_j| that fixes the next product's
// fixed-point scale, to m >= 0: the bits of non-negative doubles order like
// their values, so an integer atomic max keeps the largest whatever the order.
__device__ inline void raise_pmax(double* scal, double m) {
  atomicMax(reinterpret_cast<unsigned long long*>(scal + S_PMAX),
            (unsigned long long)__double_as_longlong(m));
}

// Row i's sum over the product's tiles from its two fixed-point words (see
// fixed_add in tiles.h): the exact integer sum, rounded once to fp64 and
// unscaled. The words are cleared for the next product.
__device__ inline double fixed_take(int64_t* acc, int64_t i, double inv_scale) {
  const int64_t L = acc[2 * i], H = acc[2 * i + 1];
  acc[2 * i] = 0;
  acc[2 * i + 1] = 0;
  const int64_t H2 = H + (L >> 32);   // L >= 0: a sum of unsigned 32-bit limbs
  const int64_t L2 = L & 0xffffffffLL;
  return ((double)H2 * 4294967296.0 + (double)L2) * inv_scale;
}

// (K p)_i of a finished product: as k_lin_rows left it, or from the tiles'
// row sums, NaN once any of its row sums was not finite.
__device__ inline double product_row(const RankOne& c, int64_t i, double inv_scale, bool bad) {
  if (c.kp) return c.kp[i];
  const double t = fixed_take(c.acc, i, inv_scale);
  return bad ? __builtin_nan("") : t;
}

// ------------------------------------------------------------- a1 layout ----
// Panel-major, feature-blocked layout. Points are grouped in panels of TP
// (the tile edge) and features in blocks of SB; panel pb holds its nkb blocks
// one after the other, each a slab of kSlabElems elements:
//   fp64: each point's SB features contiguous,
//     Xb[((pb * nkb + kb) * TP + (i % TP)) * SB + kk] = x_i[kb * SB + kk],  pb = i / TP;
//   fp32: the three bf16 slices of the values, in chunks of 8 features of one
//     point and slice, in split_chunk order.
// A tile therefore streams one contiguous run of memory per panel (few pages,
// coalesced). Zero fill beyond n points and d features.
//
// One workgroup moves one block of BK features of a panel (BK bytes x TP x
// the type's size = 16 KiB of points) as 16-byte chunks, PER per thread, all
// loads issued before the stores: chunk c is point c / CPR's features
// (c % CPR) VEC .., a piece of one input row, so the lanes of a load
// instruction read whole 128-byte row segments. With vec_ok (d a multiple of
// VEC and X 16-byte aligned) a chunk is one vector load; otherwise each
// element is loaded on its own.
template <typename T, int VEC>
__device__ inline bool load_chunk(const T* __restrict__ X, int64_t n, int64_t d, int64_t i,
                                  int64_t k, int vec_ok, T* v) {
  typedef T vec_t __attribute__((ext_vector_type(VEC)));
  vec_t x;
  if (vec_ok) {
    if (i < n && k < d) {
      x = *reinterpret_cast<const vec_t*>(X + i * d + k);
    } else {
#pragma unroll
      for (int e = 0; e < VEC; ++e) x[e] = T(0);
    }
  } else {
#pragma unroll
    for (int e = 0; e < VEC; ++e) x[e] = (i < n && k + e < d) ? X[i * d + k + e] : T(0);
  }
  bool bad = false;
#pragma unroll
  for (int e = 0; e < VEC; ++e) {
    bad |= !__builtin_isfinite(x[e]);
    v[e] = x[e];
  }
  return bad;
}

__global__ __launch_bounds__(256) void k_layout(const double* __restrict__ X, int64_t n, int64_t d,
                                                double* __restrict__ Xb, int64_t nslab, int64_t nkb,
                                                int vec_ok, int* __restrict__ flags) {
  constexpr int TP = TileShape<double>::T, BK = TileShape<double>::BK;
  constexpr int VEC = 2, CPR = BK / VEC, PER = TP * CPR / 256;
  static_assert(BK == TileShape<double>::SB && TP * CPR % 256 == 0, "one slab per workgroup");
  for (int64_t b = blockIdx.x; b < nslab; b += gridDim.x) {
    const int64_t pb = b / nkb, kb = b - pb * nkb;
    double v[PER][VEC];
    bool bad = false;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int c = u * 256 + (int)threadIdx.x;
      bad |= load_chunk<double, VEC>(X, n, d, pb * TP + c / CPR, kb * BK + (c % CPR) * VEC, vec_ok,
                                     v[u]);
    }
    double2* dst = reinterpret_cast<double2*>(Xb + b * TP * BK);
#pragma unroll
    for (int u = 0; u < PER; ++u)
      dst[u * 256 + (int)threadIdx.x] = make_double2(v[u][0], v[u][1]);
    if (bad) flags[F_NONFINITE] = 1;
  }
}

// fp32: block b of BK = 32 features is two slabs of 16; a thread takes 8
// features of a point (two vector loads) and stores them as one chunk of each
// slice (the 16 points of a quarter wave give 256 contiguous bytes).
__global__ __launch_bounds__(256) void k_layout_split(const float* __restrict__ X, int64_t n,
                                                      int64_t d, uint16_t* __restrict__ Xb,
                                                      int64_t nblk, int64_t nkb32, int vec_ok,
                                                      float scale, int check,
                                                      int* __restrict__ flags) {
  using TS = TileShape<float>;
  constexpr int TP = TS::T, CPR = TS::BK / 8, PER = TP * CPR / 256, SLAB = kSlabElems<float>;
  static_assert(TS::SB == 16 && TS::BK == 32 && TP * CPR % 256 == 0, "two slabs per block");
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  for (int64_t b = blockIdx.x; b < nblk; b += gridDim.x) {
    const int64_t pb = b / nkb32, kb = b - pb * nkb32;
    float v[PER][8];
    bool bad = false, out = false;   // out of the range the stored scale serves
    auto outside = [](float x) {
      return (fabsf(x) < kSplitMin && x != 0.f) || fabsf(x) >= kSplitMax;
    };
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int c = u * 256 + (int)threadIdx.x;
      const int64_t i = pb * TP + c / CPR, k = kb * TS::BK + (c % CPR) * 8;
      bad |= load_chunk<float, 4>(X, n, d, i, k, vec_ok, v[u]);
      bad |= load_chunk<float, 4>(X, n, d, i, k + 4, vec_ok, v[u] + 4);
    }
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int c = u * 256 + (int)threadIdx.x, p = c / CPR, q = c % CPR;
      u32x4 w[3];
#pragma unroll
      for (int e = 0; e < 8; e += 2) {
        uint16_t s0[3], s1[3];
        out |= outside(v[u][e]) || outside(v[u][e + 1]);
        bf16_split(v[u][e] * scale, s0);
        bf16_split(v[u][e + 1] * scale, s1);
#pragma unroll
        for (int t = 0; t < 3; ++t) w[t][e / 2] = (uint32_t)s0[t] | ((uint32_t)s1[t] << 16);
      }
      uint16_t* slab = Xb + (2 * b + (q >> 1)) * SLAB;
#pragma unroll
      for (int t = 0; t < 3; ++t)
        *reinterpret_cast<u32x4*>(slab + 8 * split_chunk(t, p, q & 1)) = w[t];
    }
    if (bad) flags[F_NONFINITE] = 1;
    if (out && check) flags[F_RANGE] = 1;
  }
}

__global__ __launch_bounds__(256) void k_abs_max(const float* __restrict__ X, int64_t count,
                                                 int* __restrict__ out) {
  __shared__ double sh[NT / 64];
  float m = 0.f;
  for (int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x; i < count; i += (int64_t)gridDim.x * NT)
    m = fmaxf(m, fabsf(X[i]));
  const float mx = (float)block_max((double)m, sh);
  if (threadIdx.x == 0) atomicMax(out, __float_as_int(mx));   // ordered like the values
}

// ----------------------------------------------------------- a2 norms, q ----
// VEC consecutive features of a point, from chunk c (VEC features each) of
// its row in the layout: 8 for fp32 (the three slices of a chunk summed, which
// gives the value as stored back exactly), 2 for fp64.
template <typename T> struct PointRow;
template <> struct PointRow<double> {
  static constexpr int VEC = 2, CPS = TileShape<double>::SB / VEC;   // chunks per slab row
  const double* p;
  __device__ PointRow(const double* Xb, int64_t nkb, int64_t i)
      : p(Xb + (i / TileShape<double>::T) * nkb * kSlabElems<double> +
          (i % TileShape<double>::T) * TileShape<double>::SB) {}
  __device__ void load(int64_t c, double (&v)[VEC]) const {
    const double2 x =
        *reinterpret_cast<const double2*>(p + (c / CPS) * kSlabElems<double> + (c % CPS) * VEC);
    v[0] = x.x;
    v[1] = x.y;
  }
};
template <> struct PointRow<float> {
  static constexpr int VEC = 8, CPS = TileShape<float>::SB / VEC;
  const uint16_t* p;
  int point;
  __device__ PointRow(const uint16_t* Xb, int64_t nkb, int64_t i)
      : p(Xb + (i / TileShape<float>::T) * nkb * kSlabElems<float>),
        point((int)(i % TileShape<float>::T)) {}
  __device__ void load(int64_t c, double (&v)[VEC]) const {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const uint16_t* s = p + (c / CPS) * kSlabElems<float>;
    u32x4 w[3];
#pragma unroll
    for (int t = 0; t < 3; ++t)
      w[t] = *reinterpret_cast<const u32x4*>(s + 8 * split_chunk(t, point, (int)(c % CPS)));
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      float x = 0.f;
#pragma unroll
      for (int t = 2; t >= 0; --t)
        x += bf16_value(e & 1 ? w[t][e / 2] >> 16 : w[t][e / 2] & 0xffffu);
      v[e] = (double)x;
    }
  }
};

// ||x_i||^2 and, if a pivot m is given, the cached q_i = k(x_i, x_m) for
// i < N (zero beyond) and k(x_m, x_m). fp64 sums. A workgroup takes PPB
// points, 1024 / PPB threads per point, each summing every (1024 / PPB)-th
// chunk of the point's row; the point's partial sums are then added in a fixed
// order. (256 threads left a few hundred points of many features to a few dozen
// waves: 561 x 1207 fp32 18.7 us, 502 x 2877 fp64 13.9 us; 8.7 and 9.6 us so.) The
// points of a wave's load instruction are neighbours in the layout: fp64 8 chunks
// (a whole 128-byte row) of 8 points, fp32 one chunk of 32 points (512 contiguous
// bytes per slice). Rows of up to 128 features (SHORT), which that many threads read at
// most once, take 16 (fp64) or 8 threads a point: with 64 and 32, most of them idle,
// the norms of 400000 x 30 fp64 took 84 us (20 now), norms and q of 60000 x 64 fp64 48
// us (15), of 4000 x 100 6.2 us (4.5), the norms of 50000 x 64 fp32 10.9 us (5.0);
// up to 1000 points there is no difference.
template <typename T, bool SHORT = false>
constexpr int kNormPoints = sizeof(T) == 4 ? (SHORT ? 128 : 32) : SHORT ? 64 : 16;
constexpr int kNormThreads = 1024;
template <typename T, int KER, bool SHORT>
__global__ __launch_bounds__(kNormThreads) void k_norms_q(const store_t<T>* __restrict__ Xb,
                                                          int64_t nkb, int64_t m, int64_t N,
                                                          double unscale2,
                                                          double gamma, double coef0, int degree,
                                                          T* __restrict__ norms,
                                                          double* __restrict__ q64,
                                                          double* __restrict__ scal) {
  constexpr int PPB = kNormPoints<T, SHORT>, TPP = kNormThreads / PPB, WAVES = kNormThreads / 64;
  static_assert(TileShape<T>::T % PPB == 0, "a workgroup's points lie in one panel");
  // fp64: a wave per point, or per four; fp32: a wave per two chunks of 32 points, or
  // per chunk of 64. The point's partial sums that its waves (fp32) leave:
  constexpr int PARTS = sizeof(T) == 8 ? 1 : SHORT ? TPP : WAVES;
  static_assert(sizeof(T) == 8 ? TPP == (SHORT ? 16 : 64) : TPP == (SHORT ? 8 : 2 * WAVES),
                "launch shape");
  constexpr int VEC = PointRow<T>::VEC;
  __shared__ double sh[WAVES];
  __shared__ double part[3][PARTS][PPB];
  const int tid = (int)threadIdx.x;
  const int q = sizeof(T) == 8 ? tid % TPP : tid / PPB;    // this thread's share of the chunks
  const int pl = sizeof(T) == 8 ? tid / TPP : tid % PPB;   // its point
  const int64_t i = (int64_t)blockIdx.x * PPB + pl;        // below the padded point count
  const int64_t nchunks = nkb * PointRow<T>::CPS;
  const PointRow<T> ri(Xb, nkb, i);
  double s[3] = {0.0, 0.0, 0.0};   // norm, dot, squared distance
  if (m >= 0) {
    const PointRow<T> rm(Xb, nkb, m);
#pragma unroll 4
    for (int64_t c = q; c < nchunks; c += TPP) {
      double xi[VEC], xm[VEC];
      ri.load(c, xi);
      rm.load(c, xm);
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        s[0] += xi[e] * xi[e];
        s[1] += xi[e] * xm[e];
        const double df = xi[e] - xm[e];
        s[2] += df * df;
      }
    }
  } else {
#pragma unroll 4
    for (int64_t c = q; c < nchunks; c += TPP) {
      double xi[VEC];
      ri.load(c, xi);
#pragma unroll
      for (int e = 0; e < VEC; ++e) s[0] += xi[e] * xi[e];
    }
  }
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    if (t > 0 && m < 0) break;   // uniform: the norm alone
    if constexpr (sizeof(T) == 8) {
      s[t] = SHORT ? sum_lanes(s[t], 16) : wave_sum(s[t]);
      if (q == 0) part[t][0][pl] = s[t];
    } else if constexpr (SHORT) {
      part[t][q][pl] = s[t];
    } else {
      s[t] += __shfl_xor(s[t], 32);
      if (tid % 64 < PPB) part[t][tid / 64][pl] = s[t];
    }
  }
  __syncthreads();
  double nrm = 0.0;
  if (tid < PPB) {
    double v[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      if (t > 0 && m < 0) break;
#pragma unroll
      for (int w = 0; w < PARTS; ++w) v[t] += part[t][w][tid];
      if constexpr (sizeof(T) == 4) v[t] *= unscale2;   // a power of two
    }
    nrm = v[0];
    const int64_t r = (int64_t)blockIdx.x * PPB + tid;
    norms[r] = (T)nrm;
    if (m >= 0) {
      const double kv = kernel_value64<KER>(v[1], v[2], gamma, coef0, degree);
      q64[r] = r < N ? kv : 0.0;
      if (r == m) scal[S_KMM] = kv;
    }
  }
  if (m >= 0) {   // the largest squared norm bounds the kernel values (fixed-point scale)
    const double mx = block_max(nrm, sh);
    if (tid == 0)
      atomicMax(reinterpret_cast<unsigned long long*>(scal + S_NMAX),
                (unsigned long long)__double_as_longlong(mx));
  }
}

// ------------------------------------------------------------- a3 rhs -------
template <typename T>
__global__ __launch_bounds__(256) void k_rhs_init(const T* __restrict__ y, int64_t N, int64_t NP,
                                                  double* rhs, double* x, double* xbest, double* r,
                                                  double* dir, double* bpart, int* flags,
                                                  double* scal) {
  __shared__ double sh[NT / 64];
  const double ym = (double)y[N];
  if (blockIdx.x == 0 && threadIdx.x == 0 && !(ym == 1.0 || ym == -1.0)) flags[F_BADLABEL] = 1;
  double acc = 0.0, vmax = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x; i < NP; i += (int64_t)gridDim.x * NT) {
    double v = 0.0;
    if (i < N) {
      const double yi = (double)y[i];
      if (!(yi == 1.0 || yi == -1.0)) flags[F_BADLABEL] = 1;
      v = yi - ym;
    }
    rhs[i] = v;
    x[i] = 0.0;
    xbest[i] = 0.0;
    r[i] = v;
    dir[i] = v;
    acc += v * v;
    vmax = fmax(vmax, fabs(v));
  }
  const double s = block_sum(acc, sh);
  const double mx = block_max(vmax, sh);
  if (threadIdx.x == 0) {
    bpart[blockIdx.x] = s;
    raise_pmax(scal, mx);   // the first product multiplies dir
  }
}

__global__ __launch_bounds__(256) void k_finish_delta0(const double* bpart, int64_t nb,
                                                       double* scal, double eps2,
                                                       const int* flags) {
  __shared__ double sh[NT / 64];
  const double s = sum_partials(bpart, nb, sh);
  if (threadIdx.x == 0) {
    scal[S_INFLAGS] = (flags[F_NONFINITE] ? 1.0 : 0.0) + (flags[F_BADLABEL] ? 2.0 : 0.0) +
                      (flags[F_RANGE] ? 4.0 : 0.0);
    scal[S_DELTA0] = s;
    scal[S_DHIST + 0] = s;
    double* st = scal + S_STATUS;
    st[ST_DELTA] = s;
    st[ST_CURV] = 0.0;
    st[ST_STEP] = 0.0;
    st[ST_ITER] = 0.0;
    st[ST_DONE] = s == 0.0 ? 1.0 : 0.0;   // all labels equal: alpha~ = 0 solves it
    st[ST_BREAK] = 0.0;
    st[ST_STOP] = eps2 * s;
    st[ST_STALL] = 0.0;
    scal[S_BEST] = s;     // x = 0: the residual is rhs, the energy 0
    scal[S_PHI] = 0.0;
  }
}

// ------------------------------------------------------------- a5 CG --------
// q = Q~ d from the product's row sums and the rank-one terms (zero beyond
// N), and the block partials of d^T q (c.p = d). Block 0 clears the bound on
// |p| for the next vector.
__global__ __launch_bounds__(256) void k_cg_gather(RankOne c, int64_t NP, int64_t N, double* qv,
                                                   double* bpart) {
  __shared__ double sh[NT / 64];
  if (c.scal[S_STATUS + ST_DONE] != 0.0) return;
  const RankOneSums ro = rank_one_sums(c, sh);
  const double inv = 1.0 / c.scal[S_FIXSC];
  const bool bad = c.flags[F_PRODUCT] != 0;
  double prod = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x; i < NP; i += (int64_t)gridDim.x * NT) {
    const double t = product_row(c, i, inv, bad);
    const double q = i < N ? qtilde_row(c, ro, i, t) : 0.0;
    qv[i] = q;
    prod += c.p[i] * q;
  }
  const double t = block_sum(prod, sh);
  if (threadIdx.x == 0) {
    bpart[blockIdx.x] = t;
    if (blockIdx.x == 0) c.scal[S_PMAX] = 0.0;
  }
}

// Vectors of the CG step: with CACHED, four elements of each in flight per thread
// (unrolled; restrict lets the loads move ahead of the stores), otherwise one. While
// the step's four vectors fit the Infinity Cache (256 MiB: 2^23 doubles) latency
// counts, beyond that the order in which HBM is read and written: a step with four
// and with one takes 42.7 and 45.0 us at 2 x 10^6 doubles, 125.5 and 128.1 at 2^23,
// 182.9 and 182.1 at 12 x 10^6, 250 and 241 at 16 x 10^6, 1.12 and 1.05 ms at 2^26.
// (16-byte accesses measured slower at 2^26: 4.77 against 5.25 TB/s.)
constexpr int64_t kCachedStep = int64_t(1) << 23;
template <bool CACHED> struct StepVec { using type = double* __restrict__; };
template <> struct StepVec<false> { using type = double*; };
template <bool CACHED> using step_vec = typename StepVec<CACHED>::type;
template <bool CACHED> constexpr int kStepUnroll = CACHED ? 4 : 1;

// x += a d and r -= a q (or only x += a d when the residual is about to be
// recomputed from x). On curvature breakdown (d^T q <= 0 or a step that is
// not finite) every block leaves the vectors as they are. Bound by memory.
template <bool CACHED>
__global__ __launch_bounds__(256) void k_cg_update(int x_only, const double* __restrict__ bp_in,
                                                   int64_t nb, double* scal, int par,
                                                   const double* __restrict__ dir,
                                                   const double* __restrict__ qv,
                                                   step_vec<CACHED> x, step_vec<CACHED> r,
                                                   double* bp_out, int64_t NP) {
  __shared__ double sh[NT / 64];
  if (block_stopped(scal)) return;
  const double gam = sum_partials(bp_in, nb, sh);
  const double delta = scal[S_DHIST + par];
  const double alpha = delta / gam;
  const bool broke = !(gam > 0.0) || !__builtin_isfinite(alpha);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    scal[S_ALPHA] = alpha;
    scal[S_GAMMA] = gam;
    if (broke) {
      scal[S_STATUS + ST_CURV] = gam;
      scal[S_STATUS + ST_STEP] = alpha;
      scal[S_STATUS + ST_BREAK] = 1.0;
      scal[S_STATUS + ST_DONE] = 1.0;
    }
  }
  if (broke) return;
  double v = 0.0;
  if (!x_only) {
#pragma unroll kStepUnroll<CACHED>
    for (int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x; i < NP; i += (int64_t)gridDim.x * NT) {
      x[i] = x[i] + alpha * dir[i];
      const double ri = r[i] - alpha * qv[i];
      r[i] = ri;
      v += ri * ri;
    }
    const double t = block_sum(v, sh);
    if (threadIdx.x == 0) bp_out[blockIdx.x] = t;
  } else {   // the residual recomputation multiplies x next
    for (int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x; i < NP; i += (int64_t)gridDim.x * NT) {
      const double xi = x[i] + alpha * dir[i];
      x[i] = xi;
      v = fmax(v, fabs(xi));
    }
    const double mx = block_max(v, sh);
    if (threadIdx.x == 0) raise_pmax(scal, mx);
  }
}

// r = rhs - Q~ x from the product's row sums (c.p = x), and the block
// partials of r^T r and of (rhs + r)^T x. Block 0 clears the bound on |p|.
__global__ __launch_bounds__(256) void k_cg_residual(RankOne c, int64_t NP, int64_t N,
                                                     const double* __restrict__ rhs, double* r,
                                                     double* bp_out, double* bp_phi) {
  __shared__ double sh[NT / 64];
  if (c.scal[S_STATUS + ST_DONE] != 0.0) return;
  const RankOneSums ro = rank_one_sums(c, sh);
  const double inv = 1.0 / c.scal[S_FIXSC];
  const bool bad = c.flags[F_PRODUCT] != 0;
  double v = 0.0, e = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x; i < NP; i += (int64_t)gridDim.x * NT) {
    const double t = product_row(c, i, inv, bad);
    const double ri = i < N ? rhs[i] - qtilde_row(c, ro, i, t) : 0.0;
    r[i] = ri;
    v += ri * ri;
    e += (rhs[i] + ri) * c.p[i];   // (rhs + r)^T x = -2 x (energy), zero beyond N
  }
  const double t = block_sum(v, sh);
  const double u = block_sum(e, sh);
  if (threadIdx.x == 0) {
    bp_out[blockIdx.x] = t;
    bp_phi[blockIdx.x] = u;
    if (blockIdx.x == 0) c.scal[S_PMAX] = 0.0;
  }
}

// ||rhs - Q~ x||^2 partials without touching r (final report only).
__global__ __launch_bounds__(256) void k_true_residual(RankOne c, int64_t NP, int64_t N,
                                                       const double* __restrict__ rhs,
                                                       double* bp_out) {
  __shared__ double sh[NT / 64];
  const RankOneSums ro = rank_one_sums(c, sh);
  const double inv = 1.0 / c.scal[S_FIXSC];
  const bool bad = c.flags[F_PRODUCT] != 0;
  double v = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x; i < NP; i += (int64_t)gridDim.x * NT) {
    const double t = product_row(c, i, inv, bad);
    if (i >= N) continue;
    const double ri = rhs[i] - qtilde_row(c, ro, i, t);
    v += ri * ri;
  }
  const double t = block_sum(v, sh);
  if (threadIdx.x == 0) bp_out[blockIdx.x] = t;
}

// beta = r^T r (new) / r^T r (old); d = r + beta d (beta = 0 if the old
// r^T r is 0, an exact solution). Block 0 records the iteration in the
// status (and the history) and raises done once r^T r <= eps^2 r0^T r0, and d then
// stays. raise: bound |d| for a product on tiles.
//
// At the refresh-th residual recomputation (refresh > 0) r is a true
// residual. Unless it met eps, CG has progressed if r^T r or the energy
// -(rhs + r)^T x / 2 is below the smallest so far (start and earlier
// recomputations, kept in slot (refresh - 1) & 1 of S_BEST / S_PHI; the
// updated minima go to the other slot, so no block reads a slot that block 0
// writes). A new smallest r^T r copies x to xbest; no progress at all stops
// CG, stalled, and the status then reports the best r^T r, whose iterate is
// in xbest.
//
// With `scalars` (lssvm_cg_step) block 0 also reports r^T r, d^T q, the step and
// beta there; after a breakdown, which left the vectors as they were, r^T r stays
// and beta is 0.
__global__ __launch_bounds__(256) void k_cg_direction(const double* __restrict__ bp_in, int64_t nb,
                                                      double* scal, int par, int64_t iter,
                                                      const double* __restrict__ r,
                                                      double* __restrict__ dir, int64_t NP,
                                                      double* hist, int64_t hist_cap,
                                                      int64_t refresh, int raise,
                                                      const double* __restrict__ bp_phi,
                                                      const double* __restrict__ x,
                                                      double* __restrict__ xbest,
                                                      double* __restrict__ scalars) {
  __shared__ double sh[NT / 64];
  double* st = scal + S_STATUS;
  if (block_stopped(scal)) {
    if (scalars && blockIdx.x == 0 && threadIdx.x == 0) {
      scalars[0] = scal[S_DHIST + par];
      scalars[1] = scal[S_GAMMA];
      scalars[2] = scal[S_ALPHA];
      scalars[3] = 0.0;
    }
    return;
  }
  const double dnew = sum_partials(bp_in, nb, sh);
  const double dold = scal[S_DHIST + par];
  const bool conv = dnew <= st[ST_STOP];
  bool stall = false;
  double dbest = dnew;
  if (refresh > 0 && !conv) {   // uniform over the grid: every block sums the same partials
    const double phi = -0.5 * sum_partials(bp_phi, nb, sh);
    const int rd = (int)((refresh - 1) & 1), wr = rd ^ 1;
    const double bd = scal[S_BEST + rd], bphi = scal[S_PHI + rd];
    const bool lower_res = dnew < bd, lower_phi = phi < bphi;
    stall = !lower_res && !lower_phi;
    dbest = lower_res ? dnew : bd;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      scal[S_BEST + wr] = dbest;
      scal[S_PHI + wr] = lower_phi ? phi : bphi;
    }
    if (lower_res)
      for (int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x; i < NP;
           i += (int64_t)gridDim.x * NT)
        xbest[i] = x[i];
  }
  const double beta = dold != 0.0 ? dnew / dold : 0.0;
  if (!stall && !conv) {
    double dmax = 0.0;
#pragma unroll 4
    for (int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x; i < NP;
         i += (int64_t)gridDim.x * NT) {
      const double di = r[i] + beta * dir[i];
      dir[i] = di;
      dmax = fmax(dmax, fabs(di));
    }
    if (raise) {   // the next product multiplies dir
      const double mx = block_max(dmax, sh);
      if (threadIdx.x == 0) raise_pmax(scal, mx);
    }
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    scal[S_DHIST + (par ^ 1)] = dnew;
    st[ST_DELTA] = stall ? dbest : dnew;
    st[ST_CURV] = scal[S_GAMMA];
    st[ST_STEP] = scal[S_ALPHA];
    st[ST_ITER] = (double)iter;
    if (iter <= hist_cap) hist[iter - 1] = dnew;
    if (scalars) {
      scalars[0] = dnew;
      scalars[1] = scal[S_GAMMA];
      scalars[2] = scal[S_ALPHA];
      scalars[3] = beta;   // 0 where r^T r was 0: r = 0
    }
    if (conv) st[ST_DONE] = 1.0;
    if (stall) {
      st[ST_STALL] = 1.0;
      st[ST_DONE] = 1.0;
    }
  }
}

// After r = rhs - Q~ x0 for a warm start: r^T r becomes the current delta
// (the stop threshold stays eps^2 rhs^T rhs), the direction starts at r, x0
// is the best iterate so far (with its residual and energy), and done is
// raised if x0 already meets the threshold.
__global__ __launch_bounds__(256) void k_warm_start(const double* __restrict__ bp_in,
                                                    const double* __restrict__ bp_phi, int64_t nb,
                                                    double* scal, const double* __restrict__ r,
                                                    double* dir, const double* __restrict__ x,
                                                    double* __restrict__ xbest, int64_t NP) {
  __shared__ double sh[NT / 64];
  const double dlt = sum_partials(bp_in, nb, sh);
  const double phi = -0.5 * sum_partials(bp_phi, nb, sh);
  double dmax = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x; i < NP; i += (int64_t)gridDim.x * NT) {
    dir[i] = r[i];
    xbest[i] = x[i];
    dmax = fmax(dmax, fabs(r[i]));
  }
  const double mx = block_max(dmax, sh);
  if (threadIdx.x == 0) raise_pmax(scal, mx);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    double* st = scal + S_STATUS;
    scal[S_DHIST + 0] = dlt;
    scal[S_BEST] = dlt;
    scal[S_PHI] = phi;
    st[ST_DELTA] = dlt;
    if (dlt <= st[ST_STOP]) st[ST_DONE] = 1.0;
  }
}

// ------------------------------------------------- a5 on caller vectors -----
// One CG iteration on vectors the caller holds, with q = A d supplied: the
// block partials of d^T q; block 0 also enters the caller's scalars[0] (r^T r) in
// the double-buffered slot and clears the status, with a stop threshold that no
// r^T r reaches, for the update and direction kernels, which follow.
template <bool CACHED>
__global__ __launch_bounds__(256) void k_step_dot(const double* __restrict__ a,
                                                  const double* __restrict__ b, int64_t len,
                                                  double* __restrict__ bp_out,
                                                  const double* __restrict__ scalars,
                                                  double* __restrict__ scal) {
  __shared__ double sh[NT / 64];
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    scal[S_DHIST + 0] = scalars[0];
    scal[S_DHIST + 1] = scalars[0];
    for (int k = 0; k < ST_COUNT; ++k) scal[S_STATUS + k] = 0.0;
    scal[S_STATUS + ST_STOP] = -1.0;
  }
  double v = 0.0;
#pragma unroll kStepUnroll<CACHED>
  for (int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x; i < len; i += (int64_t)gridDim.x * NT)
    v += a[i] * b[i];
  const double t = block_sum(v, sh);
  if (threadIdx.x == 0) bp_out[blockIdx.x] = t;
}

// ------------------------------------------------------------- a6 bias ------
// alpha = [x, -sum x] (last row of Eq. (11)); b = y_m + Q_mm sum x - q^T x (Eq. (15)).
template <typename T>
__global__ __launch_bounds__(1024) void k_bias(const double* __restrict__ x,
                                               const double* __restrict__ q64, int64_t N,
                                               const T* __restrict__ y, double* scal, double invC,
                                               T* __restrict__ alpha_out) {
  __shared__ double sh[1024 / 64];
  double sx = 0.0, sqx = 0.0, xmax = 0.0;
  for (int64_t i = threadIdx.x; i < N; i += blockDim.x) {
    const double xi = x[i];
    sx += xi;
    sqx += q64[i] * xi;
    xmax = fmax(xmax, fabs(xi));
    alpha_out[i] = (T)xi;
  }
  sx = block_sum(sx, sh);
  sqx = block_sum(sqx, sh);
  xmax = block_max(xmax, sh);
  if (threadIdx.x == 0) {
    scal[S_PMAX] = xmax;   // an optional true-residual product multiplies x next
    alpha_out[N] = (T)(-sx);
    const double qmm = scal[S_KMM] + invC;
    scal[S_B] = (double)y[N] + qmm * sx - sqx;
  }
}

template <typename T>
__global__ void k_single_point(const T* __restrict__ y, T* __restrict__ alpha_out, double* scal,
                               int* flags) {
  if (threadIdx.x == 0) {
    const double y0 = (double)y[0];
    const bool bad = !(y0 == 1.0 || y0 == -1.0);
    if (bad) flags[F_BADLABEL] = 1;
    if (!bad && flags[F_NONFINITE] == 0) alpha_out[0] = T(0);   // outputs untouched on error
    scal[S_B] = y0;
  }
}

// ------------------------------------------ a7 for few points: k_predict_few ----
// Decision values of up to 128 points (16 NB) on a polynomial or RBF model, from
// the caller's rows: with one tile row of test points the tile path reads the
// model once to lay it out, writes it, and reads it for the norms and for the
// tiles. Here it is read once, straight into matrix-core operands (16 x 16 x 4,
// in T: fp32 products and sums as fp32). Bound by that read up to about 64 points
// (fp64) or 32 (fp32), by the matrix cores beyond. Measured, the whole call, tile
// path before: 8192 x 512 fp64 cubic, 16 points 113 -> 41 us; 50000 x 2800 fp64
// RBF, 5 points 1310 -> 269 us (4.2 TB/s); 11490 x 3521 fp64 RBF, 89 points 733
// -> 693 us; 31219 x 2028 fp32 cubic, 76 points 281 -> 227 us; 25583 x 3000 fp32
// cubic, 128 points 356 -> 338 us.
//
// A workgroup takes blocks of 16 RB model points; its four waves share the
// features in chunks of 16 (wave v the chunks v, v + 4, ...), so that even a
// small model keeps every CU loading. Lane l holds features 4 (l / 16) .. + 3 of
// a chunk, of model point l % 16 and, from the cache, of test point l % 16 of
// each block of 16. Squared norms (RBF) are summed on the way in fp64. The
// waves' products are added in LDS in order, then 16 NB threads groups apply the
// kernel function and sum alpha_i k over the block's points in fp64; a
// workgroup's sums over its blocks are one partial per test point.
template <typename T> struct Mfma16;
template <> struct Mfma16<double> {
  using acc_t = doublex4;
  __device__ static inline acc_t mma(double a, double b, acc_t c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  __device__ static inline int row(int v, int lane) { return (lane >> 4) + 4 * v; }
};
template <> struct Mfma16<float> {
  typedef float acc_t __attribute__((ext_vector_type(4)));
  __device__ static inline acc_t mma(float a, float b, acc_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  __device__ static inline int row(int v, int lane) { return 4 * (lane >> 4) + v; }
};

// Features k .. k + 3 of a row, zero from d on; vec: 16-byte loads (d a multiple
// of the loads' width, rows aligned).
template <typename T>
__device__ inline void load4(const T* __restrict__ x, int64_t k, int64_t d, int vec, T (&v)[4]) {
  constexpr int W = 16 / (int)sizeof(T);
  typedef T vec_t __attribute__((ext_vector_type(W)));
  if (vec) {
#pragma unroll
    for (int h = 0; h < 4; h += W) {
      vec_t t;
      if (k + h < d) {
        t = *reinterpret_cast<const vec_t*>(x + k + h);
      } else {
#pragma unroll
        for (int e = 0; e < W; ++e) t[e] = T(0);
      }
#pragma unroll
      for (int e = 0; e < W; ++e) v[h + e] = t[e];
    }
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = k + e < d ? x[k + e] : T(0);
  }
}

template <typename T, int KER, int RB, int NB>
__global__ __launch_bounds__(256) void k_predict_few(PredictFew<T> a) {
  using MF = Mfma16<T>;
  constexpr int ROWS = 16 * RB, COLS = 16 * NB, GRP = NT / COLS;
  constexpr int LDG = COLS + 1;
  __shared__ T g[ROWS * LDG];
  __shared__ double nrm[2][NT / 64][ROWS > COLS ? ROWS : COLS];
  __shared__ double sums[GRP][COLS];
  const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int cl = lane & 15, kl = lane >> 4;
  const int64_t nblk = (a.n + ROWS - 1) / ROWS, nchk = (a.d + 15) / 16;
  double total = 0.0;   // of this thread's test point and share of the rows
  T finite = T(0);      // NaN once a value is not finite
  for (int64_t b = blockIdx.x; b < nblk; b += gridDim.x) {
    const T* xa[RB];
    const T* xb[NB];
#pragma unroll
    for (int r = 0; r < RB; ++r) {
      const int64_t i = b * ROWS + r * 16 + cl;
      xa[r] = a.Xtr + (i < a.n ? i : a.n - 1) * a.d;   // repeated rows get weight 0
    }
#pragma unroll
    for (int c = 0; c < NB; ++c) {
      const int64_t t = c * 16 + cl;
      xb[c] = a.Xte + (t < a.n_test ? t : a.n_test - 1) * a.d;   // repeated: not written
    }
    typename MF::acc_t acc[RB][NB];
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
      for (int c = 0; c < NB; ++c) acc[r][c] = typename MF::acc_t{};
    double na[RB] = {}, nb[NB] = {};
    for (int64_t ch = wave; ch < nchk; ch += NT / 64) {
      const int64_t k = ch * 16 + 4 * kl;
      T va[RB][4], vb[NB][4];
#pragma unroll
      for (int r = 0; r < RB; ++r) load4<T>(xa[r], k, a.d, a.vec, va[r]);
#pragma unroll
      for (int c = 0; c < NB; ++c) load4<T>(xb[c], k, a.d, a.vec, vb[c]);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int r = 0; r < RB; ++r)
#pragma unroll
          for (int c = 0; c < NB; ++c) acc[r][c] = MF::mma(va[r][e], vb[c][e], acc[r][c]);
#pragma unroll
      for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          finite += T(0) * va[r][e];
          if constexpr (KER == KRBF) na[r] += (double)va[r][e] * (double)va[r][e];
        }
#pragma unroll
      for (int c = 0; c < NB; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          finite += T(0) * vb[c][e];
          if constexpr (KER == KRBF) nb[c] += (double)vb[c][e] * (double)vb[c][e];
        }
    }
    if constexpr (KER == KRBF) {   // a point's four lanes, then the waves below
      auto lanes = [&](double v) {
        v += __shfl_xor(v, 16);
        return v + __shfl_xor(v, 32);
      };
#pragma unroll
      for (int r = 0; r < RB; ++r) {
        const double v = lanes(na[r]);
        if (kl == 0) nrm[0][wave][r * 16 + cl] = v;
      }
#pragma unroll
      for (int c = 0; c < NB; ++c) {
        const double v = lanes(nb[c]);
        if (kl == 0) nrm[1][wave][c * 16 + cl] = v;
      }
    }
    for (int w = 0; w < NT / 64; ++w) {
      if (wave == w) {
#pragma unroll
        for (int r = 0; r < RB; ++r)
#pragma unroll
          for (int c = 0; c < NB; ++c)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              T& s = g[(r * 16 + MF::row(v, lane)) * LDG + c * 16 + cl];
              s = w == 0 ? acc[r][c][v] : s + acc[r][c][v];
            }
      }
      __syncthreads();
    }
    const int c = tid % COLS, part = tid / COLS;
    double nt = 0.0;
    if constexpr (KER == KRBF)
      nt = ((nrm[1][0][c] + nrm[1][1][c]) + nrm[1][2][c]) + nrm[1][3][c];
#pragma unroll 4
    for (int r = part; r < ROWS; r += GRP) {
      const int64_t i = b * ROWS + r;
      if (i >= a.n) continue;
      double nr = 0.0;
      if constexpr (KER == KRBF)
        nr = ((nrm[0][0][r] + nrm[0][1][r]) + nrm[0][2][r]) + nrm[0][3][r];
      double kv;   // the polynomial's base and power in fp64, as on tiles
      if constexpr (KER == KPOLY) {
        const double base = a.gamma * (double)g[r * LDG + c] + a.coef0;
        kv = base;
        for (int e = 1; e < a.degree; ++e) kv *= base;
      } else {
        kv = (double)kernel_value<KER, T>(g[r * LDG + c], (T)nt, (T)nr, T(0), T(0), a.rbf_scale);
      }
      total += kv * (double)a.alpha[i];
    }
    __syncthreads();   // g and nrm are free
  }
  sums[tid / COLS][tid % COLS] = total;
  const int bad = __syncthreads_or(!(finite == T(0)));
  if (tid < COLS && tid < a.n_test) {
    double s = 0.0;
#pragma unroll
    for (int p = 0; p < GRP; ++p) s += sums[p][tid];
    a.part[(int64_t)tid * gridDim.x + blockIdx.x] = s;
  }
  if (tid == 0) a.bad[blockIdx.x] = bad;
}

// One workgroup per test point: b + the sum of its nslots partials, and the
// label, unless a workgroup met a value that is not finite (then only the flag).
template <typename T>
__global__ __launch_bounds__(256) void k_predict_few_end(const double* __restrict__ part,
                                                         const int* __restrict__ bad,
                                                         int64_t nslots, double b,
                                                         T* __restrict__ scores,
                                                         int32_t* __restrict__ labels,
                                                         int* __restrict__ flags) {
  __shared__ double sh[NT / 64];
  double s = 0.0;
  int any = 0;
  for (int64_t k = threadIdx.x; k < nslots; k += NT) {
    s += part[(int64_t)blockIdx.x * nslots + k];
    any |= bad[k];
  }
  any = __syncthreads_or(any);
  s = block_sum(s, sh);
  if (threadIdx.x != 0) return;
  if (blockIdx.x == 0) flags[F_NONFINITE] = any;
  if (any) return;
  const double f = b + s;
  scores[blockIdx.x] = (T)f;
  if (labels) labels[blockIdx.x] = f > 0.0 ? 1 : -1;
}

// ----------------------------------------- linear kernel: through w = X^T p ----
// For the linear kernel Phi is the identity, so K p = X (X^T p) and a decision
// value is <X^T alpha, x> + b (Eq. (15)): two passes over the points, O(n d),
// in place of the O(n^2 d) contraction, on the rows as the caller stores them.
// fp64 throughout (fp32 products and sums are not rounded before the result).
//
// k_lin_w: w = X^T p by chunks of rows. A workgroup takes 64 VEC columns of
// `rows` rows; a wave reads one row's 64 VEC values per load, its four waves
// every fourth row, and a thread sums its VEC columns. The four waves' sums
// are added in order and written as the chunk's partial w; k_lin_w_sum adds the
// chunks in order. Bound by the read of X (from the Infinity Cache where it
// fits). P says what p is:
//   P_VEC    a vector (fp64), S and T of the rank-one terms left per chunk;
//   P_DIR    the new CG direction r + beta d, formed here (what
//            k_cg_direction does, which saves its launch), written to dir_out;
//   P_ALPHA  model coefficients (T); X is checked for non-finite values.
enum LinP : int { P_VEC = 0, P_DIR = 1, P_ALPHA = 2 };

// Sums of the linear passes carry their rounding errors along (an unevaluated
// pair hi + lo: the exact error of a product by fma, of an addition by Knuth's
// two-sum), so K p is rounded once, at the end. Contraction stays off in them:
// an a * b merged into the additions that use p has its error counted twice
// (2e-18 of sum |a b| over 1024 terms instead of some 1e-32, more where the sum
// cancels). Ten instructions per value either way, and memory-bound.
struct Pair {
  double hi, lo;
};
__device__ inline void pair_add(Pair& s, double v) {
#pragma clang fp contract(off)
  const double t = s.hi + v, z = t - s.hi;
  s.lo += (s.hi - (t - z)) + (v - z);
  s.hi = t;
}
__device__ inline void pair_fma(Pair& s, double a, double b) {   // s += a b
#pragma clang fp contract(off)
  const double p = a * b;
  s.lo += __builtin_fma(a, b, -p);
  pair_add(s, p);
}
__device__ inline void pair_join(Pair& s, const Pair& v) {
  pair_add(s, v.hi);
  s.lo += v.lo;
}
// Sums of four pairs over a wave, reduce-scattered: the lanes of 16-lane row r
// end with the total of a[r]. Lane bits 5 and 4 halve the pairs a lane carries
// (permlane swaps), DPP moves sum the 16 lanes that are left.
__device__ inline Pair pair_swap_join(const Pair& a, const Pair& b, bool by32) {
  const uint64_t ah = as_u64(a.hi), al = as_u64(a.lo), bh = as_u64(b.hi), bl = as_u64(b.lo);
  auto swap = [&](uint64_t x, uint64_t y, double& first, double& second) {
    const auto lo = by32 ? __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)y, false, false)
                         : __builtin_amdgcn_permlane16_swap((uint32_t)x, (uint32_t)y, false, false);
    const auto hi = by32 ? __builtin_amdgcn_permlane32_swap((uint32_t)(x >> 32),
                                                            (uint32_t)(y >> 32), false, false)
                         : __builtin_amdgcn_permlane16_swap((uint32_t)(x >> 32),
                                                            (uint32_t)(y >> 32), false, false);
    first = as_f64(lo[0], hi[0]);
    second = as_f64(lo[1], hi[1]);
  };
  Pair s, o;
  swap(ah, bh, s.hi, o.hi);
  swap(al, bl, s.lo, o.lo);
  pair_join(s, o);
  return s;
}
template <int CTRL>
__device__ inline void pair_dpp_join(Pair& s) {
  const Pair o{dpp_move<CTRL>(s.hi), dpp_move<CTRL>(s.lo)};
  pair_join(s, o);
}
__device__ inline Pair pair_wave_sum4(const Pair (&a)[4]) {
  Pair s = pair_swap_join(pair_swap_join(a[0], a[2], true), pair_swap_join(a[1], a[3], true), false);
  pair_dpp_join<kDppRowHalfMirror>(s);
  pair_dpp_join<kDppQuadXor1>(s);
  pair_dpp_join<kDppQuadXor2>(s);
  pair_dpp_join<kDppRowRor8>(s);
  return s;
}
constexpr int kLinTile = 256;   // rows of p staged at a time

template <typename T, int VEC>
__device__ inline void load_vec(const T* __restrict__ x, int64_t k, int64_t d, T (&v)[VEC]) {
  if constexpr (VEC == 1) {
    v[0] = k < d ? x[k] : T(0);
  } else {
    typedef T vec_t __attribute__((ext_vector_type(VEC)));
    vec_t t;
    if (k < d) {   // d is a multiple of VEC
      t = *reinterpret_cast<const vec_t*>(x + k);
    } else {
#pragma unroll
      for (int e = 0; e < VEC; ++e) t[e] = T(0);
    }
#pragma unroll
    for (int e = 0; e < VEC; ++e) v[e] = t[e];
  }
}

template <typename T, int VEC, int P>
__global__ __launch_bounds__(256) void k_lin_w(const T* __restrict__ X, int64_t N, int64_t d,
                                               int64_t rows, LinVec v, const T* __restrict__ alpha,
                                               const double* __restrict__ q64,
                                               Pair* __restrict__ part, double* __restrict__ pq,
                                               int* __restrict__ flags) {
  __shared__ double sh[NT / 64];
  __shared__ double ps[kLinTile];
  __shared__ Pair red[NT / 64][64 * VEC];
  const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t k = ((int64_t)blockIdx.x * 64 + lane) * VEC;
  const int64_t i0 = (int64_t)blockIdx.y * rows, i1 = i0 + rows < N ? i0 + rows : N;
  // the first rows are on their way while beta is summed
  constexpr int U = 8;   // rows in flight per wave
  T x[U][VEC];
  auto load_rows = [&](int64_t r0, int cnt, int r) {
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (r + u * (NT / 64) < cnt)   // uniform over the wave
        load_vec<T, VEC>(X + (r0 + r + u * (NT / 64)) * d, k, d, x[u]);
  };
  auto tile_rows = [&](int64_t r0) { return (int)(i1 - r0 < kLinTile ? i1 - r0 : kLinTile); };
  load_rows(i0, tile_rows(i0), wave);
  double beta = 0.0;
  if constexpr (P == P_DIR) {   // this launch may raise the flag
    if (v.stop && block_stopped(v.scal)) return;
  } else if constexpr (P == P_VEC) {
    if (v.stop && v.scal[S_STATUS + ST_DONE] != 0.0) return;
  }
  if constexpr (P == P_DIR) {
    double* st = v.scal + S_STATUS;
    const double dnew = sum_partials(v.bp, v.nb, sh);
    const double dold = v.scal[S_DHIST + v.par];
    const bool conv = dnew <= st[ST_STOP];   // uniform over the grid
    if (blockIdx.x == 0 && blockIdx.y == 0 && tid == 0) {
      v.scal[S_DHIST + (v.par ^ 1)] = dnew;
      st[ST_DELTA] = dnew;
      st[ST_CURV] = v.scal[S_GAMMA];
      st[ST_STEP] = v.scal[S_ALPHA];
      st[ST_ITER] = (double)v.iter;
      if (v.iter <= v.hist_cap) v.hist[v.iter - 1] = dnew;
      if (conv) st[ST_DONE] = 1.0;
    }
    if (conv) return;
    beta = dold != 0.0 ? dnew / dold : 0.0;
  }
  Pair acc[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) acc[e] = Pair{0.0, 0.0};
  double sp = 0.0, sq = 0.0;
  bool bad = false;
  for (int64_t r0 = i0; r0 < i1; r0 += kLinTile) {
    const int cnt = tile_rows(r0);
    double pi = 0.0;
    if (tid < cnt) {
      const int64_t i = r0 + tid;
      if constexpr (P == P_ALPHA) {
        pi = (double)alpha[i];
      } else if constexpr (P == P_DIR) {
        pi = v.r[i] + beta * v.p[i];
        if (blockIdx.x == 0) v.dir_out[i] = pi;
      } else {
        pi = v.p[i];
      }
      if (P != P_ALPHA && blockIdx.x == 0) {
        sp += pi;
        sq += q64[i] * pi;
      }
    }
    if (r0 != i0) __syncthreads();   // the previous tile's readers are done
    ps[tid] = pi;
    __syncthreads();
    for (int r = wave; r < cnt; r += U * (NT / 64)) {
      if (r0 != i0 || r != wave) load_rows(r0, cnt, r);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (r + u * (NT / 64) >= cnt) continue;   // uniform over the wave
        const double pr = ps[r + u * (NT / 64)];
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
          pair_fma(acc[e], pr, (double)x[u][e]);
          if (P == P_ALPHA) bad |= !__builtin_isfinite(x[u][e]);
        }
      }
    }
  }
#pragma unroll
  for (int e = 0; e < VEC; ++e) red[wave][lane * VEC + e] = acc[e];
  __syncthreads();
  for (int c = tid; c < 64 * VEC; c += NT) {
    const int64_t col = (int64_t)blockIdx.x * 64 * VEC + c;
    Pair s = red[0][c];
#pragma unroll
    for (int w = 1; w < NT / 64; ++w) pair_join(s, red[w][c]);
    if (col < d) part[(int64_t)blockIdx.y * d + col] = s;
  }
  if (P == P_ALPHA) {
    if (bad) flags[F_NONFINITE] = 1;
  } else if (blockIdx.x == 0) {
    sp = block_sum(sp, sh);
    sq = block_sum(sq, sh);
    if (tid == 0) {
      pq[blockIdx.y] = sp;
      pq[gridDim.y + blockIdx.y] = sq;
    }
  }
}

// 64 columns per workgroup; wave v adds chunks v, v + 4, ... (eight loads in
// flight), then the four sums are added in order.
__global__ __launch_bounds__(256) void k_lin_w_sum(const Pair* __restrict__ part,
                                                   int64_t nchunks, int64_t d,
                                                   double* __restrict__ w) {
  __shared__ Pair sh[NT / 64][64];
  const int lane = (int)threadIdx.x & 63, wave = (int)threadIdx.x >> 6;
  const int64_t k = (int64_t)blockIdx.x * 64 + lane;
  Pair s{0.0, 0.0};
  if (k < d) {
#pragma unroll 8
    for (int64_t c = wave; c < nchunks; c += NT / 64) pair_join(s, part[c * d + k]);
  }
  sh[wave][lane] = s;
  __syncthreads();
  if (wave == 0 && k < d) {
#pragma unroll
    for (int v = 1; v < NT / 64; ++v) pair_join(s, sh[v][lane]);
    w[k] = s.hi;
    w[d + k] = s.lo;
  }
}

// k_lin_rows: f_i = <x_i, w> for the rows of X, four rows at a time so that a
// piece of w serves four rows: a wave takes them alone (CS = 1), or the
// workgroup's four waves take a quarter of the columns each (CS = 4: long rows
// of few points). M says where f goes:
//   R_Q       w is the pivot's row (T): q_i, k(x_m, x_m); checks X for
//             non-finite values
//   R_KP      (K p)_i into out
//   R_GATHER  (Q~ p)_i into out and the block partials of p^T Q~ p
//             (k_cg_gather on the spot)
//   R_OUT     (Q~ p)_i as T, nothing if the flags report a non-finite point
//   R_SCORE   f_i into out; checks X for non-finite values
enum LinM : int { R_Q = 0, R_KP = 1, R_GATHER = 2, R_OUT = 3, R_SCORE = 4 };
constexpr int kLinRows = 4;

template <typename T, int VEC, int CS, int M>
__global__ __launch_bounds__(256) void k_lin_rows(const T* __restrict__ X, int64_t nrows, int64_t d,
                                                  const double* __restrict__ w, int64_t m,
                                                  RankOne c, double* __restrict__ out,
                                                  T* __restrict__ outT, double* __restrict__ bp,
                                                  int* __restrict__ flags) {
  using W = typename std::conditional<M == R_Q, T, double>::type;
  __shared__ double sh[NT / 64];
  __shared__ Pair red[CS][kLinRows];
  // What the end needs from memory is read first and waited for after the rows.
  double stop = 0.0, pS = 0.0, pT = 0.0, qmm = 0.0;
  if (M == R_GATHER) stop = c.scal[S_STATUS + ST_DONE];
  if (M == R_OUT) stop = (double)flags[F_NONFINITE];
  if constexpr (M == R_GATHER || M == R_OUT) {
    for (int64_t t = threadIdx.x; t < c.nT; t += NT) {
      pS += c.pq[t];
      pT += c.pq[c.nT + t];
    }
    qmm = c.scal[S_KMM] + c.invC;
  }
  const W* wv;
  if constexpr (M == R_Q) wv = X + m * d;
  else wv = w;
  RankOneSums ro{};
  bool summed = false;
  const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
  constexpr int GROUPS = CS == 1 ? NT / 64 : 1;   // row groups per workgroup and step
  const int64_t ngroups = (nrows + kLinRows - 1) / kLinRows;
  double prod = 0.0;
  bool bad = false;
  for (int64_t g0 = (int64_t)blockIdx.x * GROUPS; g0 < ngroups; g0 += (int64_t)gridDim.x * GROUPS) {
    const int64_t g = g0 + (CS == 1 ? wave : 0), i0 = g * kLinRows;
    Pair acc[kLinRows];
    const T* x[kLinRows];
#pragma unroll
    for (int r = 0; r < kLinRows; ++r) {
      acc[r] = Pair{0.0, 0.0};
      const int64_t i = i0 + r;
      x[r] = X + (i < nrows ? i : nrows - 1) * d;   // a repeated last row is not written
    }
    if (CS > 1 || g < ngroups) {
#pragma unroll 2
      for (int64_t k = (int64_t)((CS == 1 ? 0 : wave * 64) + lane) * VEC; k < d;
           k += 64 * VEC * CS) {
        W wk[VEC], wl[VEC];
        load_vec<W, VEC>(wv, k, d, wk);
        if constexpr (M != R_Q) load_vec<W, VEC>(wv + d, k, d, wl);
        T xv[kLinRows][VEC];
#pragma unroll
        for (int r = 0; r < kLinRows; ++r) load_vec<T, VEC>(x[r], k, d, xv[r]);
#pragma unroll
        for (int r = 0; r < kLinRows; ++r)
#pragma unroll
          for (int e = 0; e < VEC; ++e) {
            pair_fma(acc[r], (double)xv[r][e], (double)wk[e]);
            if constexpr (M != R_Q) acc[r].lo += (double)xv[r][e] * wl[e];
            if (M == R_Q || M == R_SCORE) bad |= !__builtin_isfinite(xv[r][e]);
          }
      }
    }
    Pair own = pair_wave_sum4(acc);   // row i0 + lane / 16
    const int orow = lane >> 4;
    const bool finish = (lane & 15) == 0;
    if constexpr (CS > 1) {
      __syncthreads();   // the previous step's readers are done
      if (finish) red[wave][orow] = own;
      __syncthreads();
    }
    if constexpr (M == R_GATHER || M == R_OUT) {
      if (!summed) {   // uniform
        if (stop != 0.0) return;
        ro.S = block_sum(pS, sh);
        ro.Tq = block_sum(pT, sh);
        ro.qmm = qmm;
        summed = true;
      }
    }
    // one lane per row, of the group's (first) wave, finishes it
    if (finish && (CS == 1 || wave == 0)) {
      const int64_t i = i0 + orow;
      if constexpr (CS > 1) {
        own = red[0][orow];
#pragma unroll
        for (int v = 1; v < CS; ++v) pair_join(own, red[v][orow]);
      }
      double f = own.hi + own.lo;
      // a score beyond the range is the plain sum's infinity (lo is NaN there)
      if (M == R_SCORE && !__builtin_isfinite(own.hi)) f = own.hi;
      if (i < nrows) {
        if constexpr (M == R_Q) {
          if (i == m) c.scal[S_KMM] = f;
          else out[i] = f;
        } else if constexpr (M == R_KP || M == R_SCORE) {
          out[i] = f;
        } else {
          const double q = qtilde_row(c, ro, i, f);
          if constexpr (M == R_GATHER) {
            out[i] = q;
            prod += c.p[i] * q;
          } else {
            outT[i] = (T)q;
          }
        }
      }
    }
  }
  if ((M == R_Q || M == R_SCORE) && bad) flags[F_NONFINITE] = 1;
  if constexpr (M == R_GATHER) {
    const double t = block_sum(prod, sh);
    if (tid == 0) bp[blockIdx.x] = t;
  }
}

// -------------------------------------------- small linear trainings whole ----
// A whole training of the linear kernel in one workgroup, for points that fit
// its LDS (lin_train_fits): checks, q, right-hand side, CG with the stop rules
// of the separate kernels, alpha and b. An iteration is then four barriers and
// two passes over LDS instead of launches: 256 x 64 fp64 at eps 1e-10 takes
// 302 us, 4.7 us an iteration, against 723 us with a launch per iteration. Bound
// by the instructions of sixteen waves on one CU (two LDS reads and an fma per
// value, and the lane steps of six sums). Plain fp64 sums: over some hundred
// terms, in 16 parts, the pair sums of the larger problems gave the same
// iterations and errors (four shapes, 12 seeds each: 60.0 and 60.1 iterations,
// 7.7e-12 both) and took 451 us. 512 threads: 299 us here, 477 against 387 us at
// 100 x 160.
//
// w = X^T p: G lanes (a power of two, in one wave) share a column, each every
// G-th row. X w: H lanes share a row, each every H-th column; the first of them
// owns the row and keeps its x, r, direction, q and rhs in registers. ld, the
// LDS row length, spreads the lanes of both passes over the banks.
constexpr int kLinTrainThreads = 1024;
__host__ __device__ inline int lin_train_lanes(int64_t count) {   // at most 16 each
  int g = 16;
  while (g > 1 && g * count > kLinTrainThreads) g >>= 1;
  return g;
}
__host__ __device__ inline int64_t lin_train_ld(int64_t d) {
  const int64_t want = (64 / lin_train_lanes(d)) % 32;   // columns of a wave's lanes in a row
  return lin_train_lanes(d) < 4 ? d : d + (want - d % 32 + 32) % 32;
}
constexpr int64_t kLinTrainLds = 152 * 1024;

template <typename T>
__global__ __launch_bounds__(kLinTrainThreads) void k_lin_train(const T* __restrict__ X,
                                                    const T* __restrict__ y, int n, int d,
                                                    LinTrain a, T* __restrict__ alpha_out) {
  __shared__ __attribute__((aligned(16))) char lds[kLinTrainLds];
  // one reduction's wave sums each; a slot is written again only behind a barrier
  // that follows its reads (the last sums have slots of their own: CG may take none)
  __shared__ double red[9][16];
  const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6, N = n - 1;
  const int ld = (int)lin_train_ld(d), G = lin_train_lanes(d), H = lin_train_lanes(n);
  T* xs = reinterpret_cast<T*>(lds);
  double* ps = reinterpret_cast<double*>(lds + ((int64_t)n * ld * sizeof(T) + 15) / 16 * 16);
  double* w = ps + (n + 1) / 2 * 2;
  const uint64_t t_begin = wall_clock64();

  auto put = [&](int slot, double v) {   // this wave's share of a sum over the workgroup
    v = wave_sum(v);
    if (lane == 0) red[slot][wave] = v;
  };
  auto get = [&](int slot) {   // the sum, after a barrier
    double v = red[slot][lane % (kLinTrainThreads / 64)];   // 8 or 16 of them
    v += dpp_move<kDppRowHalfMirror>(v);
    v += dpp_move<kDppQuadXor1>(v);
    v += dpp_move<kDppQuadXor2>(v);
    if (kLinTrainThreads > 512) v += dpp_move<kDppRowRor8>(v);
    return v;
  };
  // X w for this thread's row, summed over its H lanes
  const int row = tid / H, h = tid % H;
  const bool owner = h == 0 && row < N;
  auto times_w = [&]() {
    double s = 0.0;
    if (row < n) {
      const T* xr = xs + row * ld;
#pragma unroll 4
      for (int c = h; c < d; c += H) {
        s += (double)xr[c] * w[c];
      }
    }
    return sum_lanes(s, H);
  };

  // ---- points, checks, q, right-hand side
  bool bad = false, bad_label = false;
  for (int k = tid; k < n * d; k += kLinTrainThreads) {
    const T v = X[k];
    bad |= !__builtin_isfinite(v);
    const int r = k / d;
    xs[r * ld + (k - r * d)] = v;
  }
  double yr = 0.0;
  const double ym = (double)y[N];
  if (row < n && h == 0) {
    yr = (double)y[row];
    bad_label = !(yr == 1.0 || yr == -1.0);
  }
  const int inflags = (__syncthreads_or(bad) ? 1 : 0) + (__syncthreads_or(bad_label) ? 2 : 0);
  for (int c = tid; c < d; c += kLinTrainThreads) w[c] = (double)xs[N * ld + c];
  __syncthreads();
  const double qi = times_w();
  if (h == 0 && row == N) red[7][0] = qi;   // k(x_m, x_m)
  const double rhs = owner ? yr - ym : 0.0;
  put(0, rhs * rhs);
  __syncthreads();
  const double kmm = red[7][0], delta0 = get(0), qmm = kmm + a.invC;
  const uint64_t t_setup = wall_clock64();

  // Q~ v for this thread's row, v a value per row; three barriers
  auto product = [&](double v) {
    if (owner) ps[row] = v;
    put(1, owner ? v : 0.0);
    put(2, owner ? qi * v : 0.0);
    __syncthreads();
    for (int c = tid / G; c < d; c += kLinTrainThreads / G) {
      double s = 0.0;
#pragma unroll 4
      for (int r = tid % G; r < N; r += G) s += ps[r] * (double)xs[r * ld + c];
      s = sum_lanes(s, G);
      if (tid % G == 0) w[c] = s;
    }
    __syncthreads();
    const double S = get(1), Tq = get(2), f = times_w();
    return owner ? f + (qmm - qi) * S - Tq + v * a.invC : 0.0;
  };

  // ---- conjugate gradients (the rules of k_cg_update and k_cg_direction)
  const double stop = a.eps2 * delta0;
  double x = 0.0, xbest = 0.0, r = rhs, dir = rhs, delta = delta0, best = delta0, phi_best = 0.0;
  double gam = 0.0, step = 0.0;
  int it = 0;
  bool broke = false, stalled = false, conv = delta0 == 0.0 || inflags != 0;
  while (!conv && it < a.max_iter) {
    const bool refresh = (it + 1) % a.replace_every == 0;
    const double q = product(dir);
    put(3, dir * q);
    __syncthreads();
    gam = get(3);
    step = delta / gam;
    if (!(gam > 0.0) || !__builtin_isfinite(step)) {
      broke = true;
      break;
    }
    x += step * dir;
    double phi = 0.0;
    if (refresh) {
      const double qx = product(x);   // every thread takes its barriers
      r = owner ? rhs - qx : 0.0;
      put(4, r * r);
      put(5, (rhs + r) * x);
      __syncthreads();
      phi = -0.5 * get(5);
    } else {
      r -= step * q;
      put(4, r * r);
      __syncthreads();
    }
    const double dnew = get(4);
    ++it;
    conv = dnew <= stop;
    double dbest = dnew;
    if (refresh && !conv) {
      const bool lower = dnew < best, lower_phi = phi < phi_best;
      stalled = !lower && !lower_phi;
      if (lower) {
        best = dnew;
        xbest = x;
      }
      if (lower_phi) phi_best = phi;
      dbest = best;
    }
    if (tid == 0 && it <= a.hist_cap) a.hist[it - 1] = dnew;
    const double beta = delta != 0.0 ? dnew / delta : 0.0;
    delta = dnew;
    if (stalled) {
      delta = dbest;
      x = xbest;
      break;
    }
    dir = r + beta * dir;
  }

  // ---- alpha_m, b (k_bias), the report
  put(6, owner ? x : 0.0);
  put(8, owner ? qi * x : 0.0);
  __syncthreads();
  const double sx = get(6), sqx = get(8);
  if (inflags == 0 && !broke) {
    if (owner) alpha_out[row] = (T)x;
    if (tid == 0) alpha_out[N] = (T)(-sx);
  }
  if (owner) {   // for a product of x afterwards
    a.x[row] = x;
    a.rhs[row] = rhs;
    a.q64[row] = qi;
  }
  if (tid < F_COUNT) a.flags[tid] = 0;
  if (tid == 0) {
    double* st = a.scal + S_STATUS;
    st[ST_DELTA] = delta;
    st[ST_CURV] = gam;
    st[ST_STEP] = step;
    st[ST_ITER] = (double)it;
    st[ST_DONE] = conv || broke || stalled ? 1.0 : 0.0;
    st[ST_BREAK] = broke ? 1.0 : 0.0;
    st[ST_STOP] = stop;
    st[ST_STALL] = stalled ? 1.0 : 0.0;
    a.scal[S_KMM] = kmm;
    a.scal[S_DELTA0] = delta0;
    a.scal[S_B] = ym + qmm * sx - sqx;
    a.scal[S_INFLAGS] = (double)inflags;
    a.scal[S_TIMES] = (double)(t_setup - t_begin);
    a.scal[S_TIMES + 1] = (double)(wall_clock64() - t_setup);
  }
}

// ------------------------------------------------------------ tile order ----
// Visit order of the upper-triangle tiles: GROUP x GROUP super-tiles column by
// column (super-rows top down), and inside each super-tile column by column.
// Position of tile (i, j) in that order: the tiles of the super-columns to
// the left, the full super-tiles above it in its super-column, and the
// columns of its super-tile before it.
__device__ inline int64_t grouped_position(int64_t nT, int64_t G, int64_t i, int64_t j) {
  const int64_t c0 = (j / G) * G, r0 = (i / G) * G;
  const int64_t ncols = (nT < c0 + G ? nT : c0 + G) - c0;
  int64_t p = c0 * (c0 + 1) / 2 + r0 * ncols;
  for (int64_t c = c0; c < j; ++c) p += (c + 1 < r0 + G ? c + 1 : r0 + G) - r0;
  return p + (i - r0);
}

// Thread t takes tile (i, j) of the column-major triangle and writes it,
// packed (i << 16) | j, at its position. The same launch zeroes the flags, the
// scalars and the row-sum words.
__global__ __launch_bounds__(256) void k_setup_clear(int64_t nT, int64_t G,
                                                     uint32_t* __restrict__ order,
                                                     int* __restrict__ flags,
                                                     double* __restrict__ scal,
                                                     int64_t* __restrict__ acc, int64_t nacc,
                                                     unsigned* __restrict__ ticket) {
  const int64_t t0 = (int64_t)blockIdx.x * NT + threadIdx.x, stride = (int64_t)gridDim.x * NT;
  if (t0 < F_COUNT) flags[t0] = 0;
  if (t0 == 0 && ticket) *ticket = 0u;
  if (t0 < S_COUNT) scal[t0] = 0.0;
  for (int64_t t = t0; t < nacc; t += stride) acc[t] = 0;
  if (!order) return;
  const int64_t W = nT * (nT + 1) / 2;
  for (int64_t t = t0; t < W; t += stride) {
    int64_t i, j;
    tri_index(t, i, j);
    order[grouped_position(nT, G, i, j)] = (uint32_t)((i << 16) | j);
  }
}

// ---------------------------------------------------------- misc vectors ----
template <typename T>
__global__ __launch_bounds__(256) void k_pad_vec(const T* __restrict__ src, int64_t len,
                                                 T* __restrict__ dst, int64_t len_pad,
                                                 const int* __restrict__ flags,
                                                 double* __restrict__ wait) {
  const int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x;
  if (i == 0) *wait = (double)flags[F_RANGE];
  if (i < len_pad) dst[i] = i < len ? src[i] : T(0);
}

template <typename T>
__global__ __launch_bounds__(256) void k_mv_out(RankOne c, int64_t NP, int64_t N,
                                                T* __restrict__ out) {
  __shared__ double sh[NT / 64];
  // out stays untouched on error, and until the points' layout stands
  if (c.flags[F_NONFINITE] != 0 || c.flags[F_RANGE] != 0) return;
  const RankOneSums ro = rank_one_sums(c, sh);
  const double inv = 1.0 / c.scal[S_FIXSC];
  const bool bad = c.flags[F_PRODUCT] != 0;
  for (int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x; i < NP; i += (int64_t)gridDim.x * NT) {
    const double t = product_row(c, i, inv, bad);
    if (i < N) out[i] = (T)qtilde_row(c, ro, i, t);
  }
}

template <typename T>
__global__ __launch_bounds__(256) void k_predict_finish(const double* __restrict__ part,
                                                        int64_t nslots, int64_t ld, int64_t n_test,
                                                        double b, T* __restrict__ scores,
                                                        int32_t* __restrict__ labels,
                                                        const int* __restrict__ flags) {
  // outputs untouched on error, and until the points' layout stands
  if (flags[F_NONFINITE] != 0 || flags[F_RANGE] != 0) return;
  // 64 test points per workgroup: wave w sums slots w, w + 4, ... (eight
  // loads in flight per lane), then the four wave sums are added in order.
  __shared__ double sh[NT / 64][64];
  const int w = (int)threadIdx.x >> 6, l = (int)threadIdx.x & 63;
  const int64_t i = (int64_t)blockIdx.x * 64 + l;
  double s = 0.0;
  if (i < n_test) {
#pragma unroll 8
    for (int64_t sl = w; sl < nslots; sl += NT / 64) s += part[sl * ld + i];
  }
  sh[w][l] = s;
  __syncthreads();
  if (w == 0 && i < n_test) {
    double f = b;
#pragma unroll
    for (int v = 0; v < NT / 64; ++v) f += sh[v][l];
    scores[i] = (T)f;
    if (labels) labels[i] = f > 0.0 ? 1 : -1;
  }
}

template <typename T>
__global__ __launch_bounds__(256) void k_pad_to_f64(const T* __restrict__ src, int64_t len,
                                                    double* __restrict__ dst, int64_t len_pad,
                                                    double* scal, const int* __restrict__ flags) {
  __shared__ double sh[NT / 64];
  const int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x;
  if (i == 0 && flags) scal[S_STATUS + ST_DONE] = (double)flags[F_RANGE];
  const double v = i < len ? (double)src[i] : 0.0;
  if (i < len_pad) dst[i] = v;
  if (scal) {   // a product multiplies dst next
    const double mx = block_max(fabs(v), sh);
    if (threadIdx.x == 0) raise_pmax(scal, mx);
  }
}

// A few doubles to pinned host memory: a copy by the stream's copy path takes
// several microseconds more than this launch.
__global__ void k_read_back(const double* __restrict__ src, int count, double* __restrict__ dst) {
  if ((int)threadIdx.x < count) dst[threadIdx.x] = src[threadIdx.x];
}

__global__ __launch_bounds__(256) void k_finish_sum(const double* bpart, int64_t nb, double* scal,
                                                    int slot) {
  __shared__ double sh[NT / 64];
  const double s = sum_partials(bpart, nb, sh);
  if (threadIdx.x == 0) scal[slot] = s;
}

// ------------------------------------------------ fused small iteration ----
// One CG iteration in one launch (launch_tiles_cg): the tiles of q = K d as
// in k_tiles, then the workgroup that finishes last does what k_cg_gather,
// k_cg_update and k_cg_direction do, for all rows at once. Each workgroup
// fences its partial sums (device-scope release) before it takes a ticket;
// the one that draws the last ticket fences again (acquire) and reads them
// all. Rows r = tid + 256 k, k < R, sit in registers: R = 4 for NP <= 1024, else 8
// (8 for all cost the small ones 3 to 6%). ONE:
// linear tiles split into single feature blocks (see tile_body). PART: whole
// tiles, or the fixup of tiles parked by a launch before.
template <typename T, int KER, int PART, bool ONE, int R>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_tiles_cg(
    TileArgs<T> a, FusedCg f) {
  if (!tile_body<T, true, KER, PART, ONE>(a)) return;   // CG had already stopped
  __shared__ int last;
  __shared__ double sh[NT / 64];
  // Every wave releases its own writes (row sums, rank-one partials) at agent
  // scope, then thread 0 draws a relaxed ticket; the workgroup that draws the
  // last one acquires before it reads. Release and acquire each on one side
  // only: full fences on both sides, and an acquire-release ticket, cost
  // ~1.8 us more per iteration.
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
  __syncthreads();
  if (threadIdx.x == 0)
    last = __hip_atomic_fetch_add(f.ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
           (unsigned)(a.ntiles - 1);
  __syncthreads();
  if (!last) return;
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  // Every global load of the vector step is issued here, at once: placed
  // where it is used, each would wait for the barrier of the reduction before
  // it and then for its own round trip, one after the other.
  const int tid = threadIdx.x;
  const RankOne& c = f.c;
  const double pS = tid < c.nT ? c.pq[tid] : 0.0;
  const double pT = tid < c.nT ? c.pq[c.nT + tid] : 0.0;
  const double kmm = f.scal[S_KMM], fxsc = f.scal[S_FIXSC];
  const double delta = f.scal[S_DHIST + f.par];
  double* st = f.scal + S_STATUS;
  const double stop = st[ST_STOP];
  const bool bad = c.flags[F_PRODUCT] != 0;
  int64_t lo[R], hi[R];
  double qm[R], dr[R], xr[R], rk[R];
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int64_t i = tid + (int64_t)k * NT;
    lo[k] = hi[k] = 0;
    qm[k] = dr[k] = xr[k] = rk[k] = 0.0;
    if (i < f.NP) {
      lo[k] = c.acc[2 * i];
      hi[k] = c.acc[2 * i + 1];
      qm[k] = i < f.N ? c.q64[i] : 0.0;
      dr[k] = f.dir[i];
      xr[k] = f.x[i];
      rk[k] = f.r[i];
    }
  }
  // S and T of the rank-one terms (one reduction for both, each summed in
  // the order of block_sum)
  double S = wave_sum(pS), Tq = wave_sum(pT);
  {
    __shared__ double sh2[2][NT / 64];
    const int w = tid >> 6;
    if ((tid & 63) == 0) {
      sh2[0][w] = S;
      sh2[1][w] = Tq;
    }
    __syncthreads();
    S = Tq = 0.0;
    for (int v = 0; v < NT / 64; ++v) {
      S += sh2[0][v];
      Tq += sh2[1][v];
    }
  }
  const double qmm = kmm + c.invC, inv = 1.0 / fxsc;
  double qr[R];
  double g = 0.0;
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int64_t i = tid + (int64_t)k * NT;
    qr[k] = 0.0;
    if (i < f.NP) {
      c.acc[2 * i] = 0;   // cleared for the next product
      c.acc[2 * i + 1] = 0;
      const int64_t H2 = hi[k] + (lo[k] >> 32);   // as fixed_take
      const double t = bad ? __builtin_nan("")
                           : ((double)H2 * 4294967296.0 + (double)(lo[k] & 0xffffffffLL)) * inv;
      const double q = i < f.N ? t + (qmm - qm[k]) * S - Tq + dr[k] * c.invC : 0.0;
      qr[k] = q;
      f.qv[i] = q;
      g += dr[k] * q;
    }
  }
  const double gam = block_sum(g, sh);
  const double alpha = delta / gam;
  if (!(gam > 0.0) || !__builtin_isfinite(alpha)) {   // curvature breakdown: nothing moves
    if (threadIdx.x == 0) {
      f.scal[S_ALPHA] = alpha;
      f.scal[S_GAMMA] = gam;
      st[ST_CURV] = gam;
      st[ST_STEP] = alpha;
      st[ST_BREAK] = 1.0;
      st[ST_DONE] = 1.0;
      *f.ticket = 0u;
    }
    return;
  }
  double rr = 0.0;
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int64_t i = tid + (int64_t)k * NT;
    if (i < f.NP) {
      f.x[i] = xr[k] + alpha * dr[k];
      rk[k] = rk[k] - alpha * qr[k];
      f.r[i] = rk[k];
      rr += rk[k] * rk[k];
    }
  }
  const double dnew = block_sum(rr, sh);
  const double beta = delta != 0.0 ? dnew / delta : 0.0;
  double dmax = 0.0;
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int64_t i = threadIdx.x + (int64_t)k * NT;
    if (i < f.NP) {
      const double di = rk[k] + beta * dr[k];
      f.dir[i] = di;
      dmax = fmax(dmax, fabs(di));
    }
  }
  dmax = block_max(dmax, sh);
  if (threadIdx.x == 0) {
    f.scal[S_PMAX] = dmax;   // the next launch multiplies dir
    f.scal[S_ALPHA] = alpha;
    f.scal[S_GAMMA] = gam;
    f.scal[S_DHIST + (f.par ^ 1)] = dnew;
    st[ST_DELTA] = dnew;
    st[ST_CURV] = gam;
    st[ST_STEP] = alpha;
    st[ST_ITER] = (double)f.iter;
    if (f.iter <= f.hist_cap) f.hist[f.iter - 1] = dnew;
    if (dnew <= stop) st[ST_DONE] = 1.0;
    *f.ticket = 0u;   // the next launch starts after this one ends
  }
}

inline unsigned blocks_for(int64_t n) { return (unsigned)((n + NT - 1) / NT); }

}  // namespace

// ------------------------------------------------------------- launchers ----

hipError_t launch_setup_clear(int64_t nT, int64_t group, uint32_t* order,
                              int* flags, double* scal, int64_t* acc, int64_t nacc,
                              unsigned* ticket, hipStream_t s) {
  const int64_t W = order ? nT * (nT + 1) / 2 : 0;
  const int64_t n = std::max<int64_t>(std::max<int64_t>(W, nacc), S_COUNT);
  const int64_t blocks = std::min<int64_t>((n + NT - 1) / NT, kVecBlocks);
  hipLaunchKernelGGL(k_setup_clear, dim3((unsigned)std::max<int64_t>(1, blocks)), dim3(NT), 0, s,
                     nT, group, order, flags, scal, acc, nacc, ticket);
  return hipGetLastError();
}

// Blocks of BK features per workgroup step (slab-stride: their count can exceed
// what one dispatch should hold).
template <>
hipError_t launch_layout<double>(const double* X, int64_t n, int64_t d, double* Xt, int64_t ld,
                                 int64_t d_pad, int, int, int* flags, hipStream_t s) {
  const int64_t nkb = d_pad / TileShape<double>::BK, nblk = (ld / TileShape<double>::T) * nkb;
  const int vec_ok = d % 2 == 0 && reinterpret_cast<uintptr_t>(X) % 16 == 0;
  const int64_t blocks = std::min<int64_t>(nblk, int64_t(1) << 20);
  hipLaunchKernelGGL(k_layout, dim3((unsigned)blocks), dim3(256), 0, s, X, n, d, Xt, nblk, nkb,
                     vec_ok, flags);
  return hipGetLastError();
}
template <>
hipError_t launch_layout<float>(const float* X, int64_t n, int64_t d, uint16_t* Xt, int64_t ld,
                                int64_t d_pad, int up, int check, int* flags,
                                hipStream_t s) {
  const int64_t nkb = d_pad / TileShape<float>::BK, nblk = (ld / TileShape<float>::T) * nkb;
  const int vec_ok = d % 4 == 0 && reinterpret_cast<uintptr_t>(X) % 16 == 0;
  const int64_t blocks = std::min<int64_t>(nblk, int64_t(1) << 20);
  hipLaunchKernelGGL(k_layout_split, dim3((unsigned)blocks), dim3(256), 0, s, X, n, d, Xt, nblk,
                     nkb, vec_ok, std::ldexp(1.f, up), check, flags);
  return hipGetLastError();
}
hipError_t launch_abs_max(const float* X, int64_t count, int* out, hipStream_t s) {
  hipLaunchKernelGGL(k_abs_max, dim3((unsigned)vec_blocks(count)), dim3(NT), 0, s, X, count, out);
  return hipGetLastError();
}

template <typename T, bool SHORT>
static hipError_t norms_q(const store_t<T>* Xt, int64_t ld, int64_t d_pad, int64_t m, int64_t N,
                          double unscale2, int kernel, double gamma, double coef0, int degree, T* norms,
                          double* q64, double* scal, hipStream_t s) {
  const int64_t nkb = d_pad / TileShape<T>::SB;
  // ld is a multiple of the tile edge
  const dim3 grid((unsigned)(ld / kNormPoints<T, SHORT>)), block(kNormThreads);
  switch (kernel) {
    case KLIN:
      hipLaunchKernelGGL((k_norms_q<T, KLIN, SHORT>), grid, block, 0, s, Xt, nkb, m, N,
                         unscale2, gamma, coef0, degree, norms, q64, scal);
      break;
    case KPOLY:
      hipLaunchKernelGGL((k_norms_q<T, KPOLY, SHORT>), grid, block, 0, s, Xt, nkb, m, N,
                         unscale2, gamma, coef0, degree, norms, q64, scal);
      break;
    default:
      hipLaunchKernelGGL((k_norms_q<T, KRBF, SHORT>), grid, block, 0, s, Xt, nkb, m, N,
                         unscale2, gamma, coef0, degree, norms, q64, scal);
      break;
  }
  return hipGetLastError();
}
template <typename T>
hipError_t launch_norms_q(const store_t<T>* Xt, int64_t ld, int64_t d_pad, int64_t m, int64_t N,
                          int up, int kernel, double gamma, double coef0, int degree, T* norms,
                          double* q64, double* scal, hipStream_t s) {
  // up to 128 features: at most one chunk per thread of 64 (fp64), half a one of 32
  constexpr int64_t kShortRow = 8;
  const double unscale2 = std::ldexp(1.0, -2 * up);
  if (d_pad / TileShape<T>::SB <= kShortRow)
    return norms_q<T, true>(Xt, ld, d_pad, m, N, unscale2, kernel, gamma, coef0, degree, norms, q64,
                            scal, s);
  return norms_q<T, false>(Xt, ld, d_pad, m, N, unscale2, kernel, gamma, coef0, degree, norms, q64,
                           scal, s);
}

// Workgroups per tile launch: 2^23 x 256 threads stays below the 2^32 work
// items one dispatch can count; a multiple of 8, so every chunk starts on XCD 0.
constexpr int64_t kMaxTileGrid = int64_t(1) << 23;

// Feature blocks per workgroup: even (the two-stage loop runs them in pairs)
// or exactly one (the single-block variant); every split holds some.
template <typename T>
inline bool blocks_ok(const TileArgs<T>& a) {
  if (a.ksplit == 1) return true;
  const int64_t per = a.split_blocks;
  return a.ksplit > 1 && (per == 1 || (per > 0 && per % 2 == 0)) && per * a.ksplit >= a.nkb &&
         per * (a.ksplit - 1) < a.nkb;
}

// Splits of a single staged block exist in fp64 only: fp32's are half a planned one.
template <typename T> constexpr bool kOneBlock = TileShape<T>::SB == TileShape<T>::BK;

template <typename T, bool SYM, int PART>
hipError_t launch_tiles(TileArgs<T> a, int kernel, int64_t nwg, hipStream_t s) {
  if (SYM && !blocks_ok(a)) return hipErrorInvalidValue;
  a.ntiles = nwg;
  for (int64_t base = 0; base < nwg; base += kMaxTileGrid) {
    a.tile_base = base;
    const dim3 grid((unsigned)std::min(kMaxTileGrid, nwg - base));
    switch (kernel) {
      case KLIN:   // whole symmetric tiles only (its splits add up, its scores need none)
        if constexpr (SYM && PART == kWhole) {
          if constexpr (kOneBlock<T>) {
            if (a.nkb == a.ksplit) {
              hipLaunchKernelGGL((k_tiles_one<T>), grid, dim3(256), 0, s, a);
              break;
            }
          }
          hipLaunchKernelGGL((k_tiles<T, SYM, KLIN, PART>), grid, dim3(256), 0, s, a);
          break;
        } else {
          return hipErrorInvalidValue;
        }
      case KPOLY:
        hipLaunchKernelGGL((k_tiles<T, SYM, KPOLY, PART>), grid, dim3(256), 0, s, a);
        break;
      default:
        hipLaunchKernelGGL((k_tiles<T, SYM, KRBF, PART>), grid, dim3(256), 0, s, a);
        break;
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <typename T>
hipError_t launch_tiles_sym(const TileArgs<T>& a, int kernel, int part, int64_t nwg,
                            hipStream_t s) {
  switch (part) {
    case kPartial: return launch_tiles<T, true, kPartial>(a, kernel, nwg, s);
    case kFixup: return launch_tiles<T, true, kFixup>(a, kernel, nwg, s);
    default: return launch_tiles<T, true, kWhole>(a, kernel, nwg, s);
  }
}

template <typename T>
hipError_t launch_tiles_gen(const TileArgs<T>& a, int kernel, int64_t nTr, hipStream_t s) {
  return launch_tiles<T, false, kWhole>(a, kernel, nTr * a.nTc, s);
}

template <typename T, int KER, int PART, bool ONE = false>
static void tiles_cg(const TileArgs<T>& a, const FusedCg& f, hipStream_t s) {
  const dim3 grid((unsigned)a.ntiles);
  if constexpr (KER != KLIN) {   // linear ones are small: kFusedMaxLinear
    if (f.NP > 4 * NT) {
      hipLaunchKernelGGL((k_tiles_cg<T, KER, PART, ONE, 8>), grid, dim3(256), 0, s, a, f);
      return;
    }
  }
  hipLaunchKernelGGL((k_tiles_cg<T, KER, PART, ONE, 4>), grid, dim3(256), 0, s, a, f);
}

template <typename T>
hipError_t launch_tiles_cg(const TileArgs<T>& a0, int kernel, int part, int64_t nwg,
                           const FusedCg& f, hipStream_t s) {
  static_assert(kFusedMaxNP <= 8 * NT && kFusedMaxLinear <= 4 * NT, "rows in registers");
  TileArgs<T> a = a0;
  a.ntiles = nwg;
  a.tile_base = 0;
  const bool fixup = part == kFixup;
  if (nwg > kMaxTileGrid || f.NP > (kernel == KLIN ? kFusedMaxLinear : kFusedMaxNP) ||
      (kernel != KLIN && !fixup && a.ksplit != 1) || (kernel == KLIN && fixup) || !blocks_ok(a))
    return hipErrorInvalidValue;
  switch (kernel) {
    case KLIN:
      if constexpr (kOneBlock<T>) {
        if (a.nkb == a.ksplit) {   // a single feature block each
          tiles_cg<T, KLIN, kWhole, true>(a, f, s);
          break;
        }
      }
      tiles_cg<T, KLIN, kWhole>(a, f, s);
      break;
    case KPOLY:
      if (fixup) tiles_cg<T, KPOLY, kFixup>(a, f, s);
      else tiles_cg<T, KPOLY, kWhole>(a, f, s);
      break;
    default:
      if (fixup) tiles_cg<T, KRBF, kFixup>(a, f, s);
      else tiles_cg<T, KRBF, kWhole>(a, f, s);
      break;
  }
  return hipGetLastError();
}

template <typename T>
hipError_t launch_rhs_init(const T* y, int64_t N, int64_t NP, double* rhs, double* x,
                           double* xbest, double* r, double* dir, double* bpart, int* flags,
                           double* scal, hipStream_t s) {
  hipLaunchKernelGGL(k_rhs_init<T>, dim3((unsigned)cg_blocks(NP)), dim3(NT), 0, s, y, N, NP, rhs,
                     x, xbest, r, dir, bpart, flags, scal);
  return hipGetLastError();
}

hipError_t launch_finish_delta0(const double* bpart, int64_t nb, double* scal, double eps2,
                                const int* flags, hipStream_t s) {
  hipLaunchKernelGGL(k_finish_delta0, dim3(1), dim3(NT), 0, s, bpart, nb, scal, eps2, flags);
  return hipGetLastError();
}

hipError_t launch_cg_gather(const RankOne& c, int64_t NP, int64_t N, double* qv, double* bpart,
                            hipStream_t s) {
  hipLaunchKernelGGL(k_cg_gather, dim3((unsigned)cg_blocks(NP)), dim3(NT), 0, s, c, NP, N, qv,
                     bpart);
  return hipGetLastError();
}

hipError_t launch_cg_update(int x_only, const double* bp_in, int64_t nb, double* scal, int par,
                            const double* dir, const double* qv, double* x, double* r,
                            double* bp_out, int64_t NP, hipStream_t s) {
  hipLaunchKernelGGL(k_cg_update<true>, dim3((unsigned)cg_blocks(NP)), dim3(NT), 0, s, x_only, bp_in,
                     nb, scal, par, dir, qv, x, r, bp_out, NP);
  return hipGetLastError();
}

hipError_t launch_cg_residual(const RankOne& c, int64_t NP, int64_t N, const double* rhs, double* r,
                              double* bp_out, double* bp_phi, hipStream_t s) {
  hipLaunchKernelGGL(k_cg_residual, dim3((unsigned)cg_blocks(NP)), dim3(NT), 0, s, c, NP, N, rhs,
                     r, bp_out, bp_phi);
  return hipGetLastError();
}

hipError_t launch_true_residual(const RankOne& c, int64_t NP, int64_t N, const double* rhs,
                                double* bp_out, hipStream_t s) {
  hipLaunchKernelGGL(k_true_residual, dim3((unsigned)cg_blocks(NP)), dim3(NT), 0, s, c, NP, N,
                     rhs, bp_out);
  return hipGetLastError();
}

hipError_t launch_cg_direction(const double* bp_in, int64_t nb, double* scal, int par,
                               int64_t iter, const double* r, double* dir, int64_t NP,
                               double* hist, int64_t hist_cap, int64_t refresh, int raise,
                               const double* bp_phi, const double* x, double* xbest,
                               hipStream_t s) {
  hipLaunchKernelGGL(k_cg_direction, dim3((unsigned)cg_blocks(NP)), dim3(NT), 0, s, bp_in, nb,
                     scal, par, iter, r, dir, NP, hist, hist_cap, refresh, raise, bp_phi, x,
                     xbest, (double*)nullptr);
  return hipGetLastError();
}

hipError_t launch_warm_start(const double* bp_in, const double* bp_phi, int64_t nb, double* scal,
                             const double* r, double* dir, const double* x, double* xbest,
                             int64_t NP, hipStream_t s) {
  hipLaunchKernelGGL(k_warm_start, dim3((unsigned)cg_blocks(NP)), dim3(NT), 0, s, bp_in, bp_phi,
                     nb, scal, r, dir, x, xbest, NP);
  return hipGetLastError();
}

// Three launches (the scalars go in and out with the first and the last). No
// bound on |d| is kept: 1024 blocks raising one word took longer than the vector
// (with the caller's product, 8 steps: 10^6 doubles 341 -> 227 us, 4 x 10^6 730 ->
// 622 us, 3 x 10^5 256 -> 154 us).
hipError_t launch_cg_step(int64_t N, double* x, double* r, double* d, const double* q,
                          double* scalars, double* scal, double* bp0, double* bp1,
                          hipStream_t s) {
  const int64_t nb = vec_blocks(N);
  const dim3 grid((unsigned)nb);
  if (N <= kCachedStep) {
    hipLaunchKernelGGL(k_step_dot<true>, grid, dim3(NT), 0, s, d, q, N, bp0, scalars, scal);
    hipLaunchKernelGGL(k_cg_update<true>, grid, dim3(NT), 0, s, 0, bp0, nb, scal, 0, d, q, x, r,
                       bp1, N);
  } else {
    hipLaunchKernelGGL(k_step_dot<false>, grid, dim3(NT), 0, s, d, q, N, bp0, scalars, scal);
    hipLaunchKernelGGL(k_cg_update<false>, grid, dim3(NT), 0, s, 0, bp0, nb, scal, 0, d, q, x, r,
                       bp1, N);
  }
  hipLaunchKernelGGL(k_cg_direction, grid, dim3(NT), 0, s, bp1, nb, scal, 0, (int64_t)1, r, d, N,
                     (double*)nullptr, (int64_t)0, (int64_t)0, 0, (const double*)nullptr,
                     (const double*)nullptr, (double*)nullptr, scalars);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_bias(const double* x, const double* q64, int64_t N, const T* y, double* scal,
                       double invC, T* alpha_out, hipStream_t s) {
  hipLaunchKernelGGL(k_bias<T>, dim3(1), dim3(1024), 0, s, x, q64, N, y, scal, invC, alpha_out);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_single_point(const T* y, T* alpha_out, double* scal, int* flags,
                               hipStream_t s) {
  hipLaunchKernelGGL(k_single_point<T>, dim3(1), dim3(64), 0, s, y, alpha_out, scal, flags);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_pad_vec(const T* src, int64_t len, T* dst, int64_t len_pad, const int* flags,
                          double* wait, hipStream_t s) {
  hipLaunchKernelGGL(k_pad_vec<T>, dim3(blocks_for(len_pad)), dim3(NT), 0, s, src, len, dst,
                     len_pad, flags, wait);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_mv_out(const RankOne& c, int64_t NP, int64_t N, T* out, hipStream_t s) {
  hipLaunchKernelGGL(k_mv_out<T>, dim3((unsigned)cg_blocks(NP)), dim3(NT), 0, s, c, NP, N, out);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_predict_finish(const double* part, int64_t nslots, int64_t ld, int64_t n_test,
                                 double b, T* scores, int32_t* labels, const int* flags,
                                 hipStream_t s) {
  hipLaunchKernelGGL(k_predict_finish<T>, dim3((unsigned)((n_test + 63) / 64)), dim3(NT), 0, s,
                     part, nslots, ld, n_test, b, scores, labels, flags);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_pad_to_f64(const T* src, int64_t len, double* dst, int64_t len_pad,
                             double* scal, const int* flags, hipStream_t s) {
  hipLaunchKernelGGL(k_pad_to_f64<T>, dim3(blocks_for(len_pad)), dim3(NT), 0, s, src, len, dst,
                     len_pad, scal, flags);
  return hipGetLastError();
}

hipError_t launch_read_back(const double* src, int count, double* dst, hipStream_t s) {
  hipLaunchKernelGGL(k_read_back, dim3(1), dim3(64), 0, s, src, count, dst);
  return hipGetLastError();
}

hipError_t launch_finish_sum(const double* bpart, int64_t nb, double* scal, int slot,
                             hipStream_t s) {
  hipLaunchKernelGGL(k_finish_sum, dim3(1), dim3(NT), 0, s, bpart, nb, scal, slot);
  return hipGetLastError();
}

// Launch shape of k_lin_w for N rows of d columns: about 512 workgroups (two
// per CU) of at least 32 rows each.
static int64_t lin_chunks_wanted(int64_t N, int64_t d, int vec) {
  const int64_t ncb = (d + 64 * vec - 1) / (64 * vec);
  return std::max<int64_t>(1, std::min<int64_t>((512 + ncb - 1) / ncb, N / 32));
}
LinShape lin_shape(int64_t N, int64_t d, int vec) {
  LinShape s;
  s.ncb = (d + 64 * vec - 1) / (64 * vec);
  const int64_t want = lin_chunks_wanted(N, d, vec);
  s.rows = (N + want - 1) / want;
  s.nch = (N + s.rows - 1) / s.rows;
  return s;
}
template <typename T>
int lin_vec(const T* X, int64_t d) {
  constexpr int V = 16 / (int)sizeof(T);
  return d % V == 0 && reinterpret_cast<uintptr_t>(X) % 16 == 0 ? V : 1;
}
// At least nch of lin_shape for N and any fewer rows: wider columns mean fewer
// column blocks, so more chunks.
int64_t lin_max_chunks(int64_t N, int64_t d) { return lin_chunks_wanted(N, d, 4); }

template <typename T, int VEC>
static hipError_t lin_w(LinP P, const T* X, int64_t N, int64_t d, const LinVec& v, const T* alpha,
                        const double* q64, double* part2, double* w, double* pq, int* flags,
                        hipStream_t s) {
  const LinShape g = lin_shape(N, d, VEC);
  Pair* part = reinterpret_cast<Pair*>(part2);
  // grid.y holds the chunks (at most 512), grid.x the column blocks
  const dim3 grid((unsigned)g.ncb, (unsigned)g.nch);
  switch (P) {
    case P_VEC:
      hipLaunchKernelGGL((k_lin_w<T, VEC, P_VEC>), grid, dim3(NT), 0, s, X, N, d, g.rows, v, alpha,
                         q64, part, pq, flags);
      break;
    case P_DIR:
      hipLaunchKernelGGL((k_lin_w<T, VEC, P_DIR>), grid, dim3(NT), 0, s, X, N, d, g.rows, v, alpha,
                         q64, part, pq, flags);
      break;
    default:
      hipLaunchKernelGGL((k_lin_w<T, VEC, P_ALPHA>), grid, dim3(NT), 0, s, X, N, d, g.rows, v,
                         alpha, q64, part, pq, flags);
      break;
  }
  hipLaunchKernelGGL(k_lin_w_sum, dim3((unsigned)((d + 63) / 64)), dim3(NT), 0, s, part, g.nch, d,
                     w);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_lin_w(const T* X, int64_t N, int64_t d, const LinVec& v, const double* q64,
                        double* part, double* w, double* pq, hipStream_t s) {
  const LinP P = v.dir_out ? P_DIR : P_VEC;
  constexpr int V = 16 / (int)sizeof(T);
  if (lin_vec(X, d) == V)
    return lin_w<T, V>(P, X, N, d, v, nullptr, q64, part, w, pq, nullptr, s);
  return lin_w<T, 1>(P, X, N, d, v, nullptr, q64, part, w, pq, nullptr, s);
}

// Workgroups of k_lin_rows: a wave per four rows, or, where that leaves fewer
// than two workgroups per CU and a row keeps four waves busy, a workgroup per
// four rows.
constexpr int64_t kLinLongRow = 512;
static bool lin_col_split(int64_t nrows, int64_t d, int vec) {
  return nrows < 16 * 512 && d >= kLinLongRow * vec;
}
static int64_t lin_row_blocks(int64_t nrows, bool split) {
  const int64_t groups = (nrows + kLinRows - 1) / kLinRows;
  return std::min<int64_t>(kVecBlocks, split ? groups : (groups + NT / 64 - 1) / (NT / 64));
}
template <typename T>
int64_t lin_gather_blocks(const T* X, int64_t N, int64_t d) {
  return lin_row_blocks(N, lin_col_split(N, d, lin_vec(X, d)));
}

template <typename T, int M>
static hipError_t lin_rows(const T* X, int64_t nrows, int64_t d, const double* w, int64_t m,
                           const RankOne& c, double* out, T* outT, double* bp, int* flags,
                           hipStream_t s) {
  constexpr int V = 16 / (int)sizeof(T);
  const int vec = lin_vec(X, d);
  const bool split = lin_col_split(nrows, d, vec);
  const dim3 grid((unsigned)lin_row_blocks(nrows, split));
  if (vec == V && split)
    hipLaunchKernelGGL((k_lin_rows<T, V, 4, M>), grid, dim3(NT), 0, s, X, nrows, d, w, m, c, out,
                       outT, bp, flags);
  else if (vec == V)
    hipLaunchKernelGGL((k_lin_rows<T, V, 1, M>), grid, dim3(NT), 0, s, X, nrows, d, w, m, c, out,
                       outT, bp, flags);
  else if (split)
    hipLaunchKernelGGL((k_lin_rows<T, 1, 4, M>), grid, dim3(NT), 0, s, X, nrows, d, w, m, c, out,
                       outT, bp, flags);
  else
    hipLaunchKernelGGL((k_lin_rows<T, 1, 1, M>), grid, dim3(NT), 0, s, X, nrows, d, w, m, c, out,
                       outT, bp, flags);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_lin_q(const T* X, int64_t n, int64_t d, double* q64, double* scal, int* flags,
                        hipStream_t s) {
  RankOne c{};
  c.scal = scal;
  return lin_rows<T, R_Q>(X, n, d, nullptr, n - 1, c, q64, nullptr, nullptr, flags, s);
}
template <typename T>
hipError_t launch_lin_kp(const T* X, int64_t N, int64_t d, const double* w, double* kp,
                         hipStream_t s) {
  return lin_rows<T, R_KP>(X, N, d, w, 0, RankOne{}, kp, nullptr, nullptr, nullptr, s);
}
template <typename T>
hipError_t launch_lin_gather(const T* X, int64_t N, int64_t d, const double* w, const RankOne& c,
                             double* qv, double* bp, hipStream_t s) {
  return lin_rows<T, R_GATHER>(X, N, d, w, 0, c, qv, nullptr, bp, nullptr, s);
}
template <typename T>
hipError_t launch_lin_out(const T* X, int64_t N, int64_t d, const double* w, const RankOne& c,
                          T* out, int* flags, hipStream_t s) {
  return lin_rows<T, R_OUT>(X, N, d, w, 0, c, nullptr, out, nullptr, flags, s);
}

bool lin_train_fits(int64_t n, int64_t d, int64_t elem) {
  if (n > kLinTrainThreads || d > kLinTrainLds) return false;
  return n * lin_train_ld(d) * elem + 16 + (n + 1) * 8 + d * 8 <= kLinTrainLds;
}
template <typename T>
hipError_t launch_lin_train(const T* X, const T* y, int64_t n, int64_t d, const LinTrain& a,
                            T* alpha_out, hipStream_t s) {
  hipLaunchKernelGGL(k_lin_train<T>, dim3(1), dim3(kLinTrainThreads), 0, s, X, y, (int)n, (int)d, a, alpha_out);
  return hipGetLastError();
}

// Partials and bad flags of k_predict_few: at most kFewBlocks workgroups.
constexpr int64_t kFewBlocks = 1024;
int64_t predict_few_slots(int64_t n, int64_t n_test) {
  const int64_t rows = n_test > 32 ? 32 : 16;
  return std::min<int64_t>(kFewBlocks, (n + rows - 1) / rows);
}
template <typename T, int KER>
static void predict_few(const PredictFew<T>& a, unsigned grid, hipStream_t s) {
  if (a.n_test > 64)
    hipLaunchKernelGGL((k_predict_few<T, KER, 2, 8>), dim3(grid), dim3(NT), 0, s, a);
  else if (a.n_test > 32)
    hipLaunchKernelGGL((k_predict_few<T, KER, 2, 4>), dim3(grid), dim3(NT), 0, s, a);
  else if (a.n_test > 16)
    hipLaunchKernelGGL((k_predict_few<T, KER, 1, 2>), dim3(grid), dim3(NT), 0, s, a);
  else
    hipLaunchKernelGGL((k_predict_few<T, KER, 1, 1>), dim3(grid), dim3(NT), 0, s, a);
}
template <typename T>
hipError_t launch_predict_few(PredictFew<T> a, int kernel, double b, T* scores, int32_t* labels,
                              int* flags, hipStream_t s) {
  if (a.n_test > kFewTests || kernel == KLIN) return hipErrorInvalidValue;
  constexpr int V = 16 / (int)sizeof(T);
  a.vec = a.d % V == 0 && reinterpret_cast<uintptr_t>(a.Xtr) % 16 == 0 &&
          reinterpret_cast<uintptr_t>(a.Xte) % 16 == 0;
  const int64_t slots = predict_few_slots(a.n, a.n_test);
  if (kernel == KPOLY) predict_few<T, KPOLY>(a, (unsigned)slots, s);
  else predict_few<T, KRBF>(a, (unsigned)slots, s);
  hipLaunchKernelGGL(k_predict_few_end<T>, dim3((unsigned)a.n_test), dim3(NT), 0, s, a.part, a.bad,
                     slots, b, scores, labels, flags);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_linear_predict(const T* Xtr, const T* alpha, int64_t n, int64_t d, const T* Xte,
                                 int64_t n_test, double b, double* part, double* w, double* f,
                                 T* scores, int32_t* labels, int* flags, hipStream_t s) {
  constexpr int V = 16 / (int)sizeof(T);
  hipError_t e =
      lin_vec(Xtr, d) == V
          ? lin_w<T, V>(P_ALPHA, Xtr, n, d, LinVec{}, alpha, nullptr, part, w, nullptr, flags, s)
          : lin_w<T, 1>(P_ALPHA, Xtr, n, d, LinVec{}, alpha, nullptr, part, w, nullptr, flags, s);
  if (e != hipSuccess) return e;
  e = lin_rows<T, R_SCORE>(Xte, n_test, d, w, -1, RankOne{}, f, nullptr, nullptr, flags, s);
  if (e != hipSuccess) return e;
  return launch_predict_finish<T>(f, 1, n_test, n_test, b, scores, labels, flags, s);
}

// ------------------------------------------------- static device scratch ----
// The working memory of lssvm_cg_step_noalloc: the scalar area and the two
// block-partial arrays of one CG vector step, at most S_COUNT + 2 (1024 + 1)
// doubles whatever the vector length (the vector kernels run at most
// kVecBlocks blocks). Every device the library runs on holds one copy until
// the process ends; calls on one device share it.
constexpr int64_t kStaticScratchDoubles = 4096;   // 32 KiB
static_assert(S_COUNT + 2 * (kVecBlocks + 1) + 64 <= kStaticScratchDoubles,
              "static scratch holds the vector step's scalars and block partials");
static __device__ __align__(256) double scratch[kStaticScratchDoubles];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double* g_scratch_ptr[kMaxDevices] = {};   // device address of `scratch`, per device
}  // namespace

// In host code `scratch` names a host-side stand-in, not device memory: the
// device address is looked up once per device (with that device current) and
// only that address is handed to kernels.
hipError_t static_scratch(double** ptr, int64_t* capacity) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = static_cast<double*>(p);
  }
  *ptr = g_scratch_ptr[dev];
  *capacity = kStaticScratchDoubles;
  return hipSuccess;
}

#define LSSVM_INSTANTIATE(T)                                                                      \
  template hipError_t launch_norms_q<T>(const store_t<T>*, int64_t, int64_t, int64_t, int64_t,    \
                                        int, int, double, double, int, T*, double*, double*,           \
                                        hipStream_t);                                             \
  template hipError_t launch_tiles_sym<T>(const TileArgs<T>&, int, int, int64_t, hipStream_t);    \
  template hipError_t launch_tiles_gen<T>(const TileArgs<T>&, int, int64_t, hipStream_t);         \
  template hipError_t launch_tiles_cg<T>(const TileArgs<T>&, int, int, int64_t, const FusedCg&,   \
                                         hipStream_t);                                            \
  template hipError_t launch_rhs_init<T>(const T*, int64_t, int64_t, double*, double*, double*,   \
                                         double*, double*, double*, int*, double*, hipStream_t);  \
  template hipError_t launch_bias<T>(const double*, const double*, int64_t, const T*, double*,    \
                                     double, T*, hipStream_t);                                    \
  template hipError_t launch_single_point<T>(const T*, T*, double*, int*, hipStream_t);           \
  template hipError_t launch_pad_vec<T>(const T*, int64_t, T*, int64_t, const int*, double*,      \
                                        hipStream_t);                                             \
  template hipError_t launch_mv_out<T>(const RankOne&, int64_t, int64_t, T*, hipStream_t);       \
  template hipError_t launch_predict_finish<T>(const double*, int64_t, int64_t, int64_t, double,  \
                                               T*, int32_t*, const int*, hipStream_t);            \
  template hipError_t launch_pad_to_f64<T>(const T*, int64_t, double*, int64_t, double*,          \
                                           const int*, hipStream_t);                                          \
  template hipError_t launch_lin_w<T>(const T*, int64_t, int64_t, const LinVec&, const double*,   \
                                      double*, double*, double*, hipStream_t);                    \
  template hipError_t launch_lin_q<T>(const T*, int64_t, int64_t, double*, double*, int*,         \
                                      hipStream_t);                                               \
  template hipError_t launch_lin_kp<T>(const T*, int64_t, int64_t, const double*, double*,        \
                                       hipStream_t);                                              \
  template hipError_t launch_lin_gather<T>(const T*, int64_t, int64_t, const double*,             \
                                           const RankOne&, double*, double*, hipStream_t);        \
  template hipError_t launch_lin_out<T>(const T*, int64_t, int64_t, const double*,                \
                                        const RankOne&, T*, int*, hipStream_t);                   \
  template int lin_vec<T>(const T*, int64_t);                                                     \
  template int64_t lin_gather_blocks<T>(const T*, int64_t, int64_t);                              \
  template hipError_t launch_predict_few<T>(PredictFew<T>, int, double, T*, int32_t*, int*,       \
                                            hipStream_t);                                         \
  template hipError_t launch_lin_train<T>(const T*, const T*, int64_t, int64_t, const LinTrain&,  \
                                          T*, hipStream_t);                                       \
  template hipError_t launch_linear_predict<T>(const T*, const T*, int64_t, int64_t, const T*,    \
                                               int64_t, double, double*, double*, double*, T*,    \
                                               int32_t*, int*, hipStream_t);

LSSVM_INSTANTIATE(float)
LSSVM_INSTANTIATE(double)

}  // namespace lssvm
