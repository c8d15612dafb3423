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

// M <= 128 rows, N columns (256 per workgroup), depth K, up to max_splits ranges.
// products: MFMA products per operand pair (1; 2: one side in two parts; 3: both).
//
// About two workgroups per CU, at least 8 chunks of 64 each. The stream wins where it
// fills the chip or where a workgroup's chain of chunks is short; with fewer workgroups
// than CUs and a long chain, a chunk's wait is not covered, and the tiled kernels, whose
// slices are half as deep, are faster. fp16 P, us, tiled / streaming:
//   rows x m -> k       16 x 8,192 -> 4,096   27 / 25     16 x 32,768 -> 2,048   90 / 108
//   64 x 32,768 -> 1,024  88 / 92 (one card)  128 x 16,384 -> 4,096  57 / 66
//   128 x 2,048 -> 2,048  14 / 12             128 x 32,768 -> 1,024  86 / 117
//   16 x 16,384 -> 8,192  71 / 66             128 x 16,384 -> 8,192  103 / 63
// Two or three products: they cover the wait, and only more than 64 rows against few
// columns that the tiled kernels take 128 at a time are slower (128 x 16,384 -> 300,
// fp32 P: 89 / 115), three products over one short range from 33 rows on (64 x 800 ->
// 300: 33 / 36).
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
    if (groups >= kCus) p.use = M > 32 || groups >= 2 * kCus || p.kc <= 2048;
    else if (M <= 32) p.use = p.kc <= 1024;
    else if (M <= 64) p.use = p.kc <= 2048;
    else p.use = p.kc <= 512 && tiles <= 8;
  } else {
    const bool narrow = round_up(N, 256) * 10 > round_up(N, 128) * 11;
    const bool slow = M > 64 ? tiles <= 4 : products == 3 && M > 32 && tiles > 1 && p.splits == 1;
    p.use = !(narrow && slow);
  }
  return p;
}

}  // namespace eogp
