// Ranges of examples that the fp16 EK-FAC squares are summed in (plain C++, no device
// code, so that a host test can check it).
#pragma once
#include <algorithm>
#include <cmath>
#include <cstdint>

#include "chip.h"

namespace eogp {

// Workgroups of one range: 128 x 128 entries each.
inline int64_t sq16_groups(int64_t d_in, int64_t d_out) { return ceil_div(d_in, 128) * ceil_div(d_out, 128); }

// Ranges of examples that a workspace always has room for.
inline int sq16_min_splits(int64_t N, int64_t d_in, int64_t d_out) {
  int64_t sp = ceil_div(2 * kCus, sq16_groups(d_in, d_out));
  sp = std::min<int64_t>(sp, std::max<int64_t>(1, N / 4));
  return (int)std::max<int64_t>(1, std::min<int64_t>(sp, 32));
}

// Time of the squares and their sum with `sp` ranges, in units of the products at full
// rounds (two workgroups per CU): the last round's empty part; a range per XCD reads its
// tokens once (a twelfth off); the partial sums written and read again at about
// 5 TB/s against the products' 0.45 PFLOP/s, 8 bytes for 2 N T operations an entry.
inline double sq16_cost(int64_t N, int64_t T, int64_t groups, int sp) {
  const double rounds = (double)(groups * sp) / (2 * kCus);
  return std::ceil(rounds) / rounds * (sp % kXcds == 0 ? 0.92 : 1.0) + 360.0 * sp / std::max<double>(1.0, (double)N * T);
}

// Example ranges of the fp16 squares when the scratch allows: eight (one XCD per
// range), or for modules whose tiles are few the multiple of eight up to 32 that
// fills the last round of two workgroups per CU best (the first at 90%), with at
// least 4 examples per range.
// More ranges where eight fill the chip cost more partial sums than the fuller round
// gives: 128 examples of 3,073 x 768 took 1,401 us with 16 ranges, 1,345 at the start;
// with eight 1,342 (1,400 at the start on that card).
// Batches of fewer than 32 examples, and modules whose tiles alone fill the chip
// (their partial sums would cost more than the shared L2 gives), take the fewest; so
// do batches of few tokens whose fewest ranges fill the chip as well (32 examples of
// 512 tokens, 2,048 x 2,048: 494 us with eight ranges, 443 with two).
inline int sq16_splits(int64_t N, int64_t T, int64_t d_in, int64_t d_out) {
  const int64_t groups = sq16_groups(d_in, d_out);
  const int least = sq16_min_splits(N, d_in, d_out);
  if (N < 32 || groups >= 2 * kCus) return least;
  int best = 8;
  double most = 0;
  for (int sp = 8; sp <= 32 && sp * 4 <= N && groups * best < 2 * kCus; sp += 8) {
    const double rounds = (double)(groups * sp) / (2 * kCus), full = rounds / std::ceil(rounds);
    if (full > most) {
      most = full;
      best = sp;
    }
    if (full >= 0.9) break;
  }
  const double rounds = (double)(groups * least) / (2 * kCus);
  const bool fills = rounds >= 0.95 * std::ceil(rounds);
  return fills && sq16_cost(N, T, groups, least) < sq16_cost(N, T, groups, best) ? least : best;
}

}  // namespace eogp
