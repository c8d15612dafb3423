// Which products of few rows stream B past a shared A (k_gemm_skinny), and how they
// split K (plain C++, no device code, so that a host test can check it).
#pragma once
#include <algorithm>
#include <cstdint>

#include "chip.h"

namespace eogp {

constexpr int64_t kSkinnyRows = 128;

struct FewRowsPlan {
  bool use;         // stream B (else the tiled kernels)
  int splits;       // ranges of K
  int64_t kc;       // K per range (multiple of 64)
};

// Whether the tiled kernels lose a round: their grid is rounded down to the XCDs, so that
// 10 units of work run on 8 workgroups (col_tiles column tiles, K in slices of 32, at least
// 16 slices a range, one round of units wanted). 128 x 2,680 -> 300: 40 us in 10 units where
// 2,048 columns in 40 units take 23.
inline bool tiled_loses_round(int64_t col_tiles, int64_t K, int max_splits) {
  const int64_t nk = ceil_div(K, (int64_t)32);
  const int64_t sp = std::max<int64_t>(1, std::min<int64_t>({(int64_t)max_splits, nk / 16, kCus / col_tiles}));
  const int64_t units = col_tiles * ceil_div(nk, ceil_div(nk, sp));
  return units > kXcds && units <= kCus && units % kXcds != 0;
}

// M <= 128 rows, N columns (256 per workgroup), depth K, up to max_splits ranges.
// products: MFMA products per operand pair (1; 2: one side in two parts; 3: both).
//
// About two workgroups per CU, at least 8 chunks of 64 each. One product, fp16 P, us, tiled /
// streaming (rows x m -> k):
// * The tiled kernels in a round too many: the stream (87 x 2,680 -> 785 37 / 23,
//   16 x 16,392 -> 12,000 202 / 125, 128 x 20,000 -> 11,264 1.25 times).
// * Fewer than 224 workgroups: a long chain of chunks is not covered, and the tiled kernels'
//   slices are half as deep (16 x 8,192 -> 4,096 27 / 25, 16 x 32,768 -> 2,048 90 / 108,
//   128 x 2,048 -> 2,048 14 / 12, 128 x 32,768 -> 1,024 86 / 117, 128 x 16,384 -> 4,096 57 / 66).
// * From there on (rows of a P a multiple of 8 KB apart share few sets of the L2, which costs
//   the tiled kernels more): 16 x 16,384 -> 8,192 71 / 66, 128 rows 103 / 63; but
//   65 x 16,392 -> 8,192 82 / 98, 65 x 8,200 -> 8,192 47 / 57.
// * More groups than CUs: the last round of the stream's counts as well, above 64 rows most
//   (128 x 20,000 -> 10,240 in 320 groups 0.68 times as fast as tiled, 128 x 16,384 -> 16,384
//   in 512 1.29 times; 16 x 32,760 -> 18,432 in 576 0.78, 48 x 20,000 -> 14,336 in 448 1.09).
// Two or three products cover the wait; only more than 64 rows against few columns that the
// tiled kernels take 128 at a time are slower (128 x 16,384 -> 300, fp32 P: 89 / 115; without
// the lost round: 65 x 2,680 -> 300 55 / 37), three products over one short range from 33 rows
// on (64 x 800 -> 300: 33 / 36).
inline FewRowsPlan few_rows_plan(int64_t M, int64_t N, int64_t K, int max_splits, int products) {
  const int64_t chunks = ceil_div(K, (int64_t)64), tiles = ceil_div(N, (int64_t)256);
  FewRowsPlan p;
  p.splits = (int)std::max<int64_t>(1, std::min<int64_t>({(int64_t)max_splits, ceil_div(2 * kCus, tiles), chunks / 8}));
  p.kc = ceil_div(chunks, (int64_t)p.splits) * 64;
  p.splits = (int)ceil_div(K, p.kc);
  const int64_t groups = tiles * p.splits;
  if (M > kSkinnyRows) {
    p.use = false;
  } else if (products == 1) {
    const bool far = K % 4096 == 0;                       // rows of P, 16-bit, 8 KB multiples apart
    const int64_t full = ceil_div(groups, (int64_t)kCus) * kCus;
    if (tiled_loses_round(tiles, K, max_splits)) p.use = true;
    else if (groups > kCus) p.use = M > 64 ? far && groups * 8 >= full * 7 : far || groups * 10 >= full * 8;
    else if (groups >= kCus * 7 / 8) p.use = far || (M <= 64 && p.kc <= 1024);
    else if (M <= 32) p.use = p.kc <= 1024;
    else if (M <= 64) p.use = p.kc <= (far ? 2048 : 1024);
    else p.use = (p.kc <= 512 && tiles <= 8) || (K < 4096 && p.kc <= 576);
  } else {
    const int64_t tiles128 = ceil_div(N, (int64_t)128);
    const bool narrow = round_up(N, 256) * 10 > tiles128 * 128 * 11;
    const bool slow = M > 64 ? tiles <= 4 && !tiled_loses_round(tiles128, K, max_splits)
                             : products == 3 && M > 32 && tiles > 1 && p.splits == 1;
    p.use = !(narrow && slow);
  }
  return p;
}

}  // namespace eogp
