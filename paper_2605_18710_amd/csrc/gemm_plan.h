// The order of a product's tiles, which tiles a weight gradient is computed in, and which of them are cut:
// host arithmetic only.
#pragma once
#include <stdint.h>
#include <stdlib.h>
#include <algorithm>

inline int64_t plan_ceil(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Tile rows (of `rows` rows each) per super-block of the tile order: the row operand of a super-block is kept to
// about half of the 256 MB last-level cache, in whole 4-row patches.  Depends on the shape alone.
#ifndef MOSAIC_LLC_ROW_BYTES
#define MOSAIC_LLC_ROW_BYTES (128 << 20)
#endif
// Only products of more than 64 x 256 rows are cut: with fewer, two rounds of 256 tiles already span every
// row and the plain order re-reads nothing that a cut would save (the weight-gradient form of the
// 7B shape, 16 tile rows, lost 3 % to a cut of 8 rows).
inline int row_block_for(int64_t K, int64_t M, int rows) {
  const int64_t tiles_m = plan_ceil(M, rows), whole = plan_ceil(tiles_m, 4) * 4;
  if (M <= 64 * 256) return (int)whole;
  const int64_t rb = (int64_t)MOSAIC_LLC_ROW_BYTES / (2 * (K > 0 ? K : 1)) / rows / 4 * 4;
  return (int)std::min<int64_t>(std::max<int64_t>(rb, 4), whole);
}

// Splitting the weight-gradient form along K.  Its contraction runs over the tokens and is
// long; its output has few tiles.  Two cases, both decided by the shape alone (256 = CUs of the
// device the kernels are written for; never the quota, so the bits stay quota-independent):
//  - up to 128 tiles of 256x256: every tile is cut, into about as many work items as CUs;
//  - more: the tiles that do not fill a round of 256 (the tail of the tile list) are cut when
//    the contraction is at least 16384 long and the cut is priced well below the alternatives,
//    one more round of large tiles or the tail as quarter tiles.  Prices in microseconds on the
//    whole device: a 256x256 tile takes 25.5 ns per unit of K, a work item 12 us on top
//    (pipeline fill, fp32 store of its piece), the pass that adds the pieces reads them at
//    3.5 TB/s after 8 us; two small workgroups per CU take 1.8 quarter units each.  Measured, pieces forced to 2 .. 8: the gate/up gradient at T=32768
//    (1376 tiles, 96 in the tail) 4845 us uncut, 4624 in 5 pieces (the plan's choice; 2 and 8
//    pieces within 15 us of it); the same at T=16384 2405 -> 2315; the down-projection gradient
//    (688 tiles, 176 in the tail, else a third round of large tiles) 2410 -> 2362 in 4 pieces
//    and slower in any other count; at T=8192 no cut gains anything (331 us either way for 96
//    tail tiles, 178 -> 211 and worse for a lone round of 192 tiles): pieces of a few thousand
//    tokens are mostly fill and drain.
// *first: first tile of the list that is cut; returns the piece count (1: nothing is cut).
inline int splitk_plan(int64_t M, int64_t N, int64_t K, int* first) {
  const int64_t t256 = plan_ceil(M, 256) * plan_ceil(N, 256);
  *first = 0;
  if (N % 4) return 1;
  if (t256 <= 128) {
    if (K < 2048) return 1;
    int64_t s = 256 / t256;
    if (s > 8) s = 8;
    while (s > 1 && plan_ceil(K, s) < 512) --s;
    return (int)s;
  }
  const int64_t tail = t256 % 256;
  if (tail == 0 || K < 16384) return 1;
  const double tile_us = 25.5e-3 * (double)K;
  int best = 1;
  double best_us = 1e30;
  for (int s = 2; s <= 8 && K / s >= 1024; ++s) {
    const double pieces = (double)(tail * s);
    const double us = (double)plan_ceil(tail * s, 256) * (tile_us / s + 12.0) + pieces * 262144.0 / 3.5e6 + 8.0;
    if (us < best_us - 1e-9) { best_us = us; best = s; }
  }
  const int64_t q = 4 * tail, full = q / 512, rem = q % 512;
  const double quarter_us = ((double)full * 2.0 * 1.8 + (rem == 0 ? 0.0 : rem <= 256 ? 1.2 * 1.8 : 2.0 * 1.8)) / 4.0 * tile_us;
  const double other_us = std::min(tile_us, quarter_us);            // one more round of large tiles, or quarter tiles
#ifdef MOSAIC_TUNING
  if (const char* e = getenv("MOSAIC_SPLITK")) { const int f = atoi(e); if (f <= 1) return 1; *first = (int)(t256 - tail); return f; }
#endif
  if (best == 1 || best_us >= 0.92 * other_us) return 1;
  *first = (int)(t256 - tail);
  return best;
}

// Weight gradients: what tiles, or pieces of tiles, of the K-strided form take on `cus` CUs, in
// microseconds.  A round's time is proportional to the contraction; nanoseconds per k-value, which rise by
// `rise` from a share `from` of the board's CUs at work to all of them (the board's power is shared), and a
// fixed part per round.  Fitted to 36 products uncut (K 128 .. 20000, 4 .. 768 tiles) and 22 cut, each on 32, 64 .. 256
// CUs, 2000 times in all: 4 % off on average, and the plan that they choose is 0.6 % slower than the
// fastest one.  The four-wave kernel is the better one only where whole rounds load the board (4608 x 4096 x 12288,
// 768 tiles on 256 CUs: 320 us, 350 with eight waves; 8192 x 2048 x 2048, 64 tiles on 64 CUs: 145 and 144).
struct RoundPrice { double ns, rise, from, fixed; };
constexpr RoundPrice kLarge8 = {16.4, 0.54, 0.52, 3.5}, kLarge4 = {16.6, 0.31, 0.60, 4.2};      // 256x256 tiles, eight and four waves
constexpr RoundPrice kPair = {11.0, 0.23, 0.30, 2.4}, kLone = {5.1, 0.35, 0.11, 1.4};           // 128x128: two to a CU (32-deep), one (64-deep)
constexpr double kFold = 1.2;                                                                   // adding a piece in registers
inline double round_us(const RoundPrice& p, double k, double busy_cus) {
  return p.fixed + k * 1e-3 * p.ns * (1.0 + p.rise * std::max(0.0, busy_cus / 256.0 - p.from) / (1.0 - p.from));
}
inline double large_us(const RoundPrice& p, double k, int64_t items, int cus) {
  const int64_t full = items / cus, rem = items % cus;
  return (double)full * round_us(p, k, cus) + (rem ? round_us(p, k, (double)rem) : 0.0);
}
// deep: K-tiles of 64 where every item has a CU to itself; folds: pieces added in registers per item
inline double small_us(double k, int64_t items, int cus, bool deep, int folds = 0) {
  const int64_t full = items / (2 * cus), rem = items % (2 * cus);
  double us = (double)full * (round_us(kPair, k, cus) + folds * kFold);
  if (rem > cus) us += kPair.fixed + (round_us(kPair, k, cus) - kPair.fixed) * (0.86 + 0.14 * (double)(rem - cus) / cus) + folds * kFold;
  else if (rem > 0) us += round_us(kLone, k * (full ? 1.05 : deep ? 1.0 : 1.24), (double)rem) + folds * kFold;
  return us;
}

// Pieces (splitk_plan) are a function of the shape; what computes them follows the quota, and every way adds
// the same pieces in the same order, so the bits do not.  Where all tiles are cut: 256x256 tiles or 128x128
// tiles with their pieces beside each other, added by a second kernel that reads them at 5 TB/s after
// 4 us, or 128x128 tiles whose pieces follow one another in one workgroup.
// Measured, pieces of 256x256 tiles -> plan, on 256, 192, 128, 64 CUs:
//   8192 x 2048 x 2048   78 101 95 176 -> 74 99 95 176      9216 x 1024 x 1024   38 37 37 61 -> 32 37 37 61
//   9216 x 1024 x 4096  83 108 103 192 -> 81 107 103 192    9216 x 1024 x 3072   70 93 88 158 -> 69 68 88 158
//   24000 x 240 x 1280    62 62 61 63 -> 30 30 44 62        9216 x 600 x 1024    35 35 35 58 -> 27 27 35 51
//   2048 x 1024 x 2048    28 28 28 44 -> 22 21 21 32        12000 x 1280 x 5120  150 235 221 428 -> 151 208 223 430
// Fewer pieces, chosen for 256 CUs, take less there and on few CUs (the first of these 71, 149, 143, 144), but leave
// the shares between them idle.
// Uncut: 256x256 tiles, 128x128 tiles, or whole rounds of large tiles and the rest in quarters.
enum WgradWay { kPiecesLarge, kPiecesSmall, kPiecesChained, kWhole8, kWhole4, kWholeSmall, kMixed8, kMixed4 };
struct WgradPlan {
  int pieces, first, kper;     // tiles from `first` on are cut into `pieces` pieces of kper k-values (splitk_plan)
  WgradWay way;                // of the cut tiles if all are cut, else of the tiles before `first`
  double us;                   // its price, without what every launch costs (only where first == 0)
};
inline WgradPlan wgrad_plan(int64_t M, int64_t N, int64_t K, int cus, bool may_cut, bool four_wave) {
  const int64_t t256 = plan_ceil(M, 256) * plan_ceil(N, 256), t128 = plan_ceil(M, 128) * plan_ceil(N, 128);
  WgradPlan p = {1, 0, 0, kWhole8, 0.0};
  if (may_cut) p.pieces = splitk_plan(M, N, K, &p.first);
  if (p.pieces > 1) p.kper = (int)(plan_ceil(plan_ceil(K, 32), p.pieces) * 32);
  if (p.pieces > 1 && p.first == 0) {
    const bool deep = p.kper % 64 == 0;
    const double add_us = 4.0 + p.pieces * (double)M * (double)N * 4.0 / 5.0e6;
    const double us[] = {large_us(kLarge8, p.kper, t256 * p.pieces, cus) + add_us, small_us(p.kper, t128 * p.pieces, cus, deep) + add_us,
                         small_us((double)K, t128, cus, deep, p.pieces - 1)};
    p.way = (WgradWay)(kPiecesLarge + (std::min_element(us, us + 3) - us));
    p.us = *std::min_element(us, us + 3);
    return p;
  }
  const int64_t tiles = p.pieces > 1 ? p.first : t256, quarters = p.pieces > 1 ? 4 * tiles : t128, head = tiles / cus * cus, rest = tiles - head;
  const bool mixed = head > 0 && rest > 0;
  const double never = 1e30, quarter_us = 5.4 + small_us((double)K, 4 * rest, cus, true);
  const double us[] = {large_us(kLarge8, (double)K, tiles, cus), four_wave ? large_us(kLarge4, (double)K, tiles, cus) : never,
                       small_us((double)K, quarters, cus, true), mixed ? large_us(kLarge8, (double)K, head, cus) + quarter_us : never,
                       mixed && four_wave ? large_us(kLarge4, (double)K, head, cus) + quarter_us : never};
  p.way = (WgradWay)(kWhole8 + (std::min_element(us, us + 5) - us));
  p.us = *std::min_element(us, us + 5);
  return p;
}

// The two products of a linear layer's backward pass, dX[T,k] = dY W^T and dW[k,n] = X^T dY, as one launch of 128x128
// tiles (64-deep K-tiles, one workgroup per CU): `wgs_d` workgroups walk the tiles of the first, `wgs_w` those of the
// second, wgs_d + wgs_w <= cus.  Small products leave most of the chip idle one after the other (1568 x 768 x 768: 78 tiles,
// then 36) and pay for two launches; side by side the longer one hides the shorter.  The tiles of a product are
// the ones that its own launch would compute, in the same order of additions (a gradient that is cut has its
// pieces chained), so the bits are those of two launches.
// Priced against the two launches with the figures above (input gradients: those of the K-strided form, and lower
// tiles of the four-wave kernel); a launch more costs kLaunchUs.  The tiles of 64 rows that an input gradient of its own may take
// (launch_mfma_shape) are not priced: pairs are chosen as if it took 128 rows, up to a fifth slower than it is there.
constexpr double kLaunchUs = 3.0;
struct PairPlan { bool pair; int wgs_d, wgs_w; double us, apart_us; };
inline PairPlan pair_plan(int64_t T, int64_t k, int64_t n, int cus, const WgradPlan& w) {
  PairPlan p = {false, 0, 0, 1e30, 0.0};
  if (cus < 16 || w.first > 0 || (w.pieces > 1 && w.kper % 64)) return p;
  const int64_t nd = plan_ceil(T, 128) * plan_ceil(k, 128), nw = plan_ceil(k, 128) * plan_ceil(n, 128);
  if (nd + nw > 8 * (int64_t)cus) return p;           // the large tiles' ground
  const double busy = (double)std::min<int64_t>(cus, nd + nw);
  const double td = round_us(kLone, (double)n, busy), tw = round_us(kLone, (double)T, busy) + (w.pieces - 1) * kFold;
  for (int g = 8; g + 8 <= cus / 8 * 8; g += 8) {
    const double us = std::max((double)plan_ceil(nd, g) * td, (double)plan_ceil(nw, cus / 8 * 8 - g) * tw);
    if (us < p.us - 1e-9) { p.us = us; p.wgs_d = g; p.wgs_w = cus / 8 * 8 - g; }
  }
  p.wgs_d = (int)std::min<int64_t>(p.wgs_d, plan_ceil(nd, 8) * 8);
  p.wgs_w = (int)std::min<int64_t>(p.wgs_w, plan_ceil(nw, 8) * 8);
  double apart = small_us((double)n, nd, cus, true);
  if (n % 64 == 0 && n >= 128) {
    const double round[] = {2.57, 2.8, 3.15, 3.5};    // of 160, 192, 224, 256 rows, as in launch_mfma_shape
    for (int i = 0; i < 4; ++i) {
      const int64_t tiles = plan_ceil(T, 160 + 32 * i) * plan_ceil(k, 256);
      apart = std::min(apart, large_us(kLarge4, (double)n, tiles, cus) * round[i] / 3.5);
    }
  }
  p.apart_us = apart + w.us + kLaunchUs;
  p.pair = p.us < 0.95 * p.apart_us;
  return p;
}
