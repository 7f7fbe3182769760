// Tile choice of the bf16 MFMA products (host only, no HIP).
#pragma once

#include <algorithm>

namespace tx {

// Output tiles of the bf16 kernels: the ring kernel's, the pair kernel's
// 128x128 (two blocks per CU) and the persistent kernel's 256x256.
enum GemmTile { T32x32, T32x64, T64x64, T64x128, T128x128, kPair, kPersistent, kGemmTiles };

constexpr int kRingK = 64;            // k columns per step of every kernel
constexpr int PT = 256, PK = kRingK;  // the persistent kernel's tile

// Estimated time of a launch: its rounds of blocks over the CUs, each a fixed
// part (prologue and epilogue, us) and a part per k step, or the rate at which
// the L2s deliver operands to all CUs (21.5 MB per us), whichever is more. A
// round that fills the chip takes longer than one of few blocks (operands are
// shared, the clock falls), so the last round lies between the two by its fill;
// the pair kernel's is of one block per CU up to half. Small tiles spread few rows
// over more CUs, large ones read less per flop; of two pair blocks on a CU one
// runs while the other waits, which pays when the tiles fill many rounds of a
// product that is none of the persistent kernel's.
// Fitted to 1185 products (32 to 140000 rows, N and K of 128 to 8192, operands
// rotating through six sets): the chosen tile is 0.8% off the fastest on average,
// 6% in 95 of 100 and 19% at most, and more than 3% behind the persistent kernel
// (where it applies, the pair kernel elsewhere) in 9. The estimates (an empty
// launch's 2 us added) are within 17% in nine of ten. Inside a call, where other
// kernels' data fill the caches, a launch takes up to a third longer.
struct TileCost {
  int bm, bn, per_cu;
  double few_fix, few_step;    // few blocks on the chip
  double full_fix, full_step;  // a full round
};
static const TileCost kTileCost[kGemmTiles] = {
    {32, 32, 1, 1.73, 0.0848, 1.50, 0.0965}, {32, 64, 1, 1.58, 0.110, 1.39, 0.112},
    {64, 64, 1, 1.59, 0.0985, 1.17, 0.209},  {64, 128, 1, 4.46, 0.0938, 2.98, 0.362},
    {128, 128, 1, 1.70, 0.320, 6.14, 0.541}, {128, 128, 2, 5.95, 1.09, 6.51, 1.18},
    {PT, PT, 1, 4.55, 0.986, 8.61, 1.33}};
constexpr double kL2MBPerUs = 21.5, kSecondLaunchUs = 5.0;

inline double tile_us(int c, int M, int N, int K, int n_cu) {
  const TileCost& t = kTileCost[c];
  const long long tiles = (long long)((M + t.bm - 1) / t.bm) * (N / t.bn), slots = (long long)n_cu * t.per_cu;
  const double steps = K / kRingK, few = t.few_fix + t.few_step * steps, full = t.full_fix + t.full_step * steps;
  const long long rounds = tiles / slots, rest = tiles % slots;
  double us = rounds * full;
  if (rest > 0) {
    const double fill = t.per_cu == 1 ? (double)rest / n_cu : std::max(0.0, (double)rest / n_cu - 1.0);
    us += few + (full - few) * fill;
  }
  return std::max(us, t.few_fix + tiles * (t.bm + t.bn) * 2.0 * K / (kL2MBPerUs * 1e6));
}

constexpr int kPersistentRows = 2048;  // below, its launch covers too few of the CUs

// Products the persistent kernel takes: N a multiple of the tile, K of two k
// steps and at least four, enough rows, element offsets within int32 (ld_max:
// the longest row).
inline bool persistent_shape(int M, int N, int K, long long ld_max) {
  return N % PT == 0 && K % (2 * PK) == 0 && K >= 4 * PK && M >= kPersistentRows && (long long)M * ld_max < (1ll << 31) &&
         (long long)N * K < (1ll << 31);
}

inline int pick_tile(int M, int N, int K, bool persistent, int n_cu, double* us = nullptr) {
  int best = kPair;
  double best_us = 1e30;
  // the ring kernel's weight offsets, as the persistent kernel's, are 32-bit
  // byte offsets
  const bool wide = (long long)N * K >= (1ll << 31);
  for (int c = 0; c < kGemmTiles; ++c) {
    if (c == kPersistent ? !persistent : wide && c != kPair) continue;
    const double t = tile_us(c, M, N, K, n_cu);
    // of small tiles within 3% the smaller: inside a call its loads, spread over
    // more CUs, wait less (one user's call 97.6 us, 99.8 without)
    if (t < (c <= T64x64 ? 0.97 : 1.0) * best_us) best_us = t, best = c;
  }
  if (us) *us = best_us;
  return best;
}

// Rows that the persistent kernel takes of a product of M: all, or those of its
// full rounds over the CUs when the rows left over run faster in a launch of
// smaller tiles than in a round that leaves most CUs idle. The estimate charges
// 5 us for the second launch (its start waits for the first one's last blocks),
// so that ties stay whole. 66500 rows, N 1024 (4.06 rounds): K 1024 151 us
// whole, 133 split, K 4096 507 and 443; 33000 rows, N 512, K 2048 93 and 71.
// Over 240 products of 1 to 9 rounds the choice is 0.1% off the better one on
// average and at most 4% behind the whole launch. Rows split off are as many as
// the kernel takes (a round of a wide output may have fewer: those stay whole).
inline int persistent_rows(int M, int N, int K, int n_cu) {
  const int tiles_n = N / PT;
  const long long tiles = (long long)((M + PT - 1) / PT) * tiles_n, rounds = tiles / n_cu;
  const long long m1 = rounds * n_cu / tiles_n * PT;
  if (rounds < 1 || tiles % n_cu == 0 || m1 < kPersistentRows || m1 >= M) return M;
  double rest = 0.0;
  pick_tile((int)(M - m1), N, K, false, n_cu, &rest);
  return tile_us(kPersistent, (int)m1, N, K, n_cu) + rest + kSecondLaunchUs < tile_us(kPersistent, M, N, K, n_cu)
             ? (int)m1
             : M;
}

}  // namespace tx
