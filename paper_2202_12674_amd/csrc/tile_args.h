// The tile kernel's interface: the kernel functions, the tile shapes, the
// XCD count and the arguments of one launch. Shared by the tile kernel
// (tiles.h) and the host runtime; measurements of the tile kernel are tied to
// this header and tiles.h.
#pragma once

#include <cstdint>

namespace lssvm {

enum Kern : int { KLIN = 0, KPOLY = 1, KRBF = 2 };

// Points per tile edge and features per staged block, per element type
// (compile-time, like the block sizes of Sec. III-C4). The symmetric schedule
// needs square tiles.
//
// Plans and padding count blocks of BK features; the kernel stages SB features
// at a time. fp64 stages its blocks whole. fp32 points are stored as three
// bf16 slices h + m + l (bf16_split in tiles.h), which hold every bit of the
// value, and the kernel multiplies the slices on the bf16 matrix cores: a
// staged block is SLICES x T x SB slice elements, 12 KiB for 16 features, so
// that two stages of two panels leave room for two workgroups on a CU.
constexpr int kNumXcd = 8;

template <typename T> struct TileShape;
template <> struct TileShape<float> {
  static constexpr int T = 128, BK = 32, SB = 16, SLICES = 3;
  using store_t = uint16_t;   // bf16 bits
};
template <> struct TileShape<double> {
  static constexpr int T = 128, BK = 16, SB = 16, SLICES = 1;
  using store_t = double;
};
// Elements of one staged block of a panel of T points.
template <typename T>
constexpr int kSlabElems = TileShape<T>::SLICES * TileShape<T>::T * TileShape<T>::SB;
template <typename T> using store_t = typename TileShape<T>::store_t;

// What a symmetric tile launch computes: whole tiles, parked feature splits
// of tiles (their raw inner products), or the fixup that sums a tile's parked
// splits and finishes it.
enum TilePart : int { kWhole = 0, kPartial = 1, kFixup = 2 };

template <typename T>
struct TileArgs {
  const store_t<T>* A;   // panel-major feature-blocked row points (see k_layout)
  const store_t<T>* B;   // panel-major feature-blocked column points
  int64_t nkb;   // staged feature blocks of SB (even)
  const T* nA;   // squared norms of row points (RBF)
  const T* nB;   // squared norms of column points (RBF)
  const double* pv;   // symmetric mode: the vector multiplied (fp64), zero beyond N
  const double* q64;  // symmetric mode: q_i = k(x_i, x_m), zero beyond N
  double* pq;         // symmetric mode: per panel I, sum p_j at [I], sum q_j p_j at [nTc + I]
  const T* wB;        // general mode: per-column weights (alpha)
  T gscale;   // fp32: what the stored points' inner products are multiplied by, a power
              // of two (they are stored scaled up: k_layout_split)
  T gamma, coef0;
  double gamma64, coef64;   // fp32 polynomial: its kernel values are formed in fp64
  T rbf_scale;   // RBF exponent scale: gamma (fp64, exp) or gamma log2(e) (fp32, exp2)
  int degree;
  int64_t nTc;   // column tiles (general mode); tiles per side (symmetric mode)
  int64_t ksplit;  // symmetric mode: workgroups per tile, split ks over the staged blocks
                   // [ks split_blocks, (ks + 1) split_blocks) below nkb. Linear kernel,
                   // whole tiles: every split adds its share of the row and column sums
                   // (the kernel value is the inner product itself). Split launches
                   // park inner products in gpart instead and a fixup launch finishes
                   // each tile.
  int64_t split_blocks;   // even, or 1 (k_tiles_one)
  int64_t tile_offset;  // symmetric mode: first tile of the launch in the visit order
  T* gpart;             // split launches: parked inner products, ksplit 128^2 per tile
  const uint32_t* order;  // symmetric mode: (I << 16) | J per visit slot, or null
  double* part;  // general mode: partial sums, part[slot * part_ld + row]
  // symmetric mode: each row's sum over tiles, in fixed point (see fixed_add):
  // acc[2 row] the low 32-bit limbs, acc[2 row + 1] the signed high limbs
  int64_t* acc;
  // symmetric mode: fx[0] = max |p_j|, fx[1] = max ||x_i||^2 (the bounds of the
  // fixed-point scale); fx[2] receives the scale 2^s the launch used
  double* fx;
  int* fx_bad;          // symmetric mode: raised when a row sum is not finite
  const double* stop;   // nonzero: the launch returns at once, as CG has stopped or as the
                        // points have to be laid out anew first (F_RANGE). Or null.
  int64_t part_ld;
  // A product's tiles may outnumber one launch (the dispatch grid counts work
  // items in 32 bits), so the launcher splits them into chunks: workgroup b of
  // a chunk takes tile slot tile_base + b of ntiles.
  int64_t tile_base, ntiles;
};

}  // namespace lssvm
