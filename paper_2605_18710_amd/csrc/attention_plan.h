// How the attention kernels' tiles are dealt to workgroups, and where a key tile's dK and dV take two groups of waves.  Host code without
// the device's headers, so that a test can compile it alone.
#pragma once
#include <algorithm>
#include <cstdint>

// Head size 128: two groups of waves to a key tile where there is at most one tile to a CU, so that the longest tile is what the
// kernel takes and a wave has its SIMD to itself (2040 cycles a block for 1024 of matrix work).  A function of the shape: the
// two groups' sums are added, so the bits follow it.  Eight waves in step do 10 to 15 % less than two workgroups of four on a CU, which
// tells where a share of the board has three and more tiles to a CU: with more tiles than half the CUs of the board the groups
// wait for long items of unequal length, a causal mask and four or more query heads to a key head.  Measured on masked streams,
// whole backward pass in us, one group -> two, on 256, 192, 128, 96, 64, 32 CUs:
//   B4 N1024 H16 Hkv4 causal (128 tiles)  236 230 238 271 331 470 -> 181 174 182 211 259 506
//   B1 N1024 H16 causal (128)             82 83 82 90 112 141 -> 72 72 72 85 101 174
//   B2 N1024 H8, no mask (128)            81 82 82 . 111 . -> 71 72 71 . 120 .
//   B4 N2048 H16 Hkv2 causal (128)        777 806 841 919 1017 2036 -> 555 578 615 682 814 1602
//   B5 N1024 H16 Hkv4 causal (160)        242 240 299 308 442 656 -> 187 185 207 246 349 635
//   B6 N1024 H32 Hkv4 causal (192)        459 468 588 598 749 1379 -> 351 359 401 492 732 1412
//   B7 N1024 H16 Hkv4 causal (224)        255 302 339 440 551 863 -> 202 212 260 349 478 880
//   B8 N1024 H16 Hkv4 causal (256)        258 322 338 385 472 916 -> 207 230 267 373 509 997
//   B2 N2048 H32 Hkv8 causal (256)        462 496 599 920 791 1550 -> 356 376 430 613 831 1645
//   B1 N4096 H32 Hkv8 causal (256)        866 980 980 1725 1947 2749 -> 653 755 770 1069 1481 2935
inline bool dkv_in_parts(int64_t items, int64_t query_tiles, int group, bool causal) {
  return query_tiles >= 8 && (items <= 128 || (items <= 256 && causal && group >= 4));
}

// The queue or static rounds, the heads whose tiles a block of the item list holds, and the consecutive items that go to one XCD.
// The queue pays once every workgroup draws several items (tiles of unequal cost under a causal mask, ragged last tiles, and
// heads that stay together on an XCD: measured 5-10 % on the audio encoder's full attention at 32 and 64 CUs, 25-40 % on causal
// rows of 4096); with up to three rounds static rounds do as well without the claims.  Its blocks: about two rounds of an XCD's
// workgroups under a causal mask, else one head.
// Not so with one workgroup to a CU (two groups of waves) and a causal mask: nothing runs beside a workgroup that got two long tiles, and
// from the second round on the queue hands out all tiles longest first, every eighth one to an XCD (with a multiple of eight heads:
// whole heads).  B1 N4096 H32 Hkv8 on 192
// CUs, backward in us: rounds 1175, this 755; B2 N2048 on 192 591, 376; B8 N768 H16 Hkv4 on 128 266, 182; with blocks of two rounds B5 N1024
// H16 Hkv4 on 128 CUs 235, 207, on 32 670, 635, B3 N1600 H40 Hkv5 on 128 684, 585 (B8 N1024 H16 Hkv4 on 32 991, 997).  Two rounds of whole heads
// are even by themselves, the second one mirrored: B1 N1024 H16 on 64 CUs 101, queue 105.
struct AttnDeal { bool queue; int hb, unit; };
inline AttnDeal attn_deal(int64_t heads, int tiles, int64_t resident, bool causal, bool one_per_cu) {
  const int64_t items = heads * tiles, per_xcd = (resident + 7) / 8;
  if (causal && one_per_cu && items > resident) {
    const bool even = items == 2 * resident && resident % 8 == 0 && resident / 8 % tiles == 0;
    return {!even, (int)heads, 1};
  }
  const int64_t two_rounds = std::max<int64_t>(1, (2 * per_xcd + tiles - 1) / tiles);
  const int hb = causal ? (int)std::min<int64_t>(two_rounds, std::max<int64_t>(1, heads / 8)) : 1;
  return {items > 3 * resident, hb, hb * tiles};
}
