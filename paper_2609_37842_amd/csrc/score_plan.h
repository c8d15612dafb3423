// How a scoring call runs: queries per pass, block size, module ranges, grid and
// workspace (plain C++, no device code, so that a host test can check it).
#pragma once
#include <algorithm>
#include <cstddef>
#include <cstdint>

#include "chip.h"

namespace eogp {

constexpr int QB = 16;                 // queries of a group (one MFMA operand)
constexpr int NW = 8;                  // waves per workgroup of the scoring pass
constexpr int SB = 64;                 // bytes of a row per step
constexpr int FRAGS = 16;              // plane fragments (1 KB) per step and 16 queries
constexpr int MSPLIT = 16;             // first-level merge workgroups per query
constexpr int MAX_RNG = 64;            // module ranges of the multi-module pass
constexpr int FOLD_ROWS = 64;          // rows per block of the fold

struct ModInfo {
  int32_t k;       // bits of the module
  int32_t coff;    // first coordinate of the module in a query row
  int32_t boff;    // first byte of the module in a code row
  int32_t sbase;   // first step of the module
};

// Queries per pass / 16 (nqt) and 32-row tiles per wave (rt).
struct PassCfg {
  int nqt, rt;
};

struct ScoreLayout {
  int64_t n_steps = 0;   // steps over all modules
  int64_t n_groups = 0;  // groups of 16 queries
  int64_t grid = 0;      // workgroups of the scoring pass
  int64_t fold_grid = 0; // workgroups of the multi-module fold (0: one module)
  int n_rng = 1;         // module ranges of the multi-module pass
  bool n64 = false;      // dots need 64 bits
  int merge_split = 1;   // first-level merge workgroups per query
  size_t o_mods = 0, o_fq = 0, o_ys = 0, o_pl = 0, o_ck = 0, o_ci = 0, o_ck2 = 0, o_ci2 = 0,
         o_part = 0,
         total = 0;
};

// Fold lists: 256 candidate slots per query when that leaves room for at least
// 128 new entries after a prune, else 512.
inline int fold_cap(int32_t topk) { return topk <= 128 ? 256 : 512; }

inline int64_t row_blocks(int64_t N, int rt) { return ceil_div(N, NW * 32 * rt); }

// A schedule of the multi-module pass: module ranges, and its length in steps of
// two-tile blocks.
struct RangePick {
  int n_rng;
  double steps;
};

// Module ranges for blocks of rt tiles per wave: the count that gives the shortest
// schedule, rounds of units (range, block) times the steps of a range (a uniform
// estimate), plus a step per unit for its start and its dots. A step of four tiles
// per wave takes 1.75 times one of two (48 modules of 8,192 bits, one round of 240
// units: 16 queries 2.4 and 4.3 us, 32 queries 3.8 and 6.6 us).
inline RangePick pick_ranges(int64_t N, int rt, int U, int64_t n_steps) {
  const int64_t n_blocks = std::max<int64_t>(1, row_blocks(N, rt));
  const double weight = rt == 4 ? 1.75 : 1.0;
  RangePick best{1, 1e300};
  const int most = (int)std::min<int64_t>({(int64_t)U, (int64_t)MAX_RNG,
                                           std::max<int64_t>(1, ceil_div(8 * kCus, n_blocks))});
  for (int r = 1; r <= most; ++r) {
    const double rounds = (double)ceil_div(n_blocks * r, kCus);
    const double steps = ((double)n_steps / U * (double)ceil_div(U, r) + 1.0) * weight;
    if (rounds * steps < best.steps * 0.999) best = RangePick{r, rounds * steps};
  }
  return best;
}

inline ScoreLayout score_layout(int64_t N, int64_t Q, int32_t U, const int64_t* kmod, int32_t topk, PassCfg c) {
  ScoreLayout L;
  int64_t kmax = 0;
  for (int u = 0; u < U; ++u) {
    L.n_steps += ceil_div(kmod[u], 8 * SB);
    kmax = std::max<int64_t>(kmax, kmod[u]);
  }
  L.n_groups = ceil_div(Q, QB);
  const int64_t n_blocks = row_blocks(N, c.rt);
  int64_t lists = 0;
  if (U == 1) {
    L.grid = std::max<int64_t>(1, std::min<int64_t>(n_blocks, kCus));
    // lists for the two-tile blocks, whichever block size runs
    lists = std::max<int64_t>(1, std::min<int64_t>(row_blocks(N, 2), kCus));
  } else {
    // one workgroup per unit, up to the CUs, and as many on each XCD as its share
    // of the units (rounded down to a multiple of the XCDs, a grid for one round
    // took two: 112 modules of 8,192 bits, 5,000 codes, 16 queries 414 -> 284 us;
    // a workgroup past its XCD's share finds no unit and ends)
    L.n_rng = pick_ranges(N, c.rt, U, L.n_steps).n_rng;
    const int64_t units = std::max<int64_t>(1, n_blocks * L.n_rng);
    L.grid = units < kXcds ? units : std::min<int64_t>(round_up(units, kXcds), kCus);
    L.fold_grid = std::max<int64_t>(1, std::min<int64_t>(ceil_div(N, FOLD_ROWS), 2 * kCus));
    lists = L.fold_grid;
  }
  L.n64 = kmax > (1 << 16);     // |n| <= k 2^14 fits 32 bits up to k = 2^16
  const size_t nq = (size_t)c.nqt * QB;
  size_t b = 0;
  auto add = [&](size_t x) { size_t o = b; b = align256(b + x); return o; };
  L.o_mods = add(sizeof(ModInfo) * U);
  L.o_fq = add(4 * (size_t)L.n_groups * U * QB);
  L.o_ys = add(8 * (size_t)L.n_groups * U * QB);
  L.o_pl = add((size_t)(L.n_groups * L.n_steps) * FRAGS * 1024);
  L.o_ck = add((size_t)lists * nq * topk * 8);
  L.o_ci = add((size_t)lists * nq * topk * 4);
  L.merge_split = (int)std::min<int64_t>(MSPLIT, std::max<int64_t>(1, lists / 8));
  L.o_ck2 = add((size_t)L.merge_split * nq * topk * 8);
  L.o_ci2 = add((size_t)L.merge_split * nq * topk * 4);
  L.o_part = add(U > 1 ? (size_t)U * nq * (size_t)N * (L.n64 ? 8 : 4) : 0);
  add(16);             // unused; the no-allocation entry's limit counts it
  L.total = b;
  return L;
}

// Queries per pass and tiles per wave.
// 32 queries per pass (nqt = 2) whenever there are more than 16: a pass then
// reads the store and expands its bits once for twice the MFMAs (1,048,576 codes
// of 16,384 bits: 0.79 ms per 32 queries against 0.89 ms per 16 before). Not for
// top-k over 128 (32 lists of more than 256 slots do not fit LDS beside the
// planes), for dots in 64 bits, nor where the workspace is too small for it:
// its candidate lists and dots are twice as many, so `ws_bytes` that hold the
// 16-query layout only get the 16-query pass, with the same results.
// Four tiles per wave (1,024-row blocks) halve the fragment reads per MFMA and
// the planes read per code byte (4,194,304 codes, 16 queries: the pass 2.5 -> 1.9
// ms with it and the requests that run on across blocks); two (512 rows) where
// the blocks' last round would be emptier. One module: rounds x (rows + a fixed
// part of a block). Several modules: the shorter schedule of the two (2 modules
// of 8,192 bits, 60,000 codes, 16 queries: 151 us with four tiles in two rounds, 94
// with two in one; 48 modules, 20,000 codes: 368 and 334 us). Row-major stores
// always two: their rows' lines are fetched again before they are used up when
// twice as many are in flight (32 modules of 5,120 bits, 197,784 codes, one
// query: 1,933 us with four tiles, 1,524 with two).
inline PassCfg choose_cfg(int64_t N, int64_t Q, int32_t U, const int64_t* kmod, int32_t topk, bool tiled,
                          size_t ws_bytes) {
  int64_t kmax = 0, n_steps = 0;
  for (int u = 0; u < U; ++u) {
    kmax = std::max<int64_t>(kmax, kmod[u]);
    n_steps += ceil_div(kmod[u], 8 * SB);
  }
  const bool n64 = kmax > (1 << 16);
  PassCfg c;
  c.rt = 2;
  c.nqt = Q > QB && topk <= 128 && !n64 ? 2 : 1;
  if (c.nqt == 2 && score_layout(N, Q, U, kmod, topk, c).total > ws_bytes) c.nqt = 1;
  if (n64 || !tiled) return c;
  if (U == 1) {
    auto rounds = [&](int rt) { return (double)ceil_div(std::max<int64_t>(1, row_blocks(N, rt)), kCus); };
    if (rounds(4) * 4.2 < rounds(2) * 2.4) c.rt = 4;
  } else if (pick_ranges(N, 4, U, n_steps).steps < pick_ranges(N, 2, U, n_steps).steps) {
    c.rt = 4;
  }
  return c;
}

// Module ranges of the multi-module pass: n_rng consecutive ranges of
// roughly equal step counts, each at least one module (one pass over the
// module sizes, no host allocation).
inline void module_ranges(const int64_t* kmod, int U, int64_t n_steps, int n_rng, int32_t* rng) {
  auto steps = [&](int u) { return ceil_div(kmod[u], 8 * SB); };
  rng[0] = 0;
  int v = 1;                   // candidate start of the next range
  int64_t base = steps(0);     // first step of module v
  for (int r = 1; r < n_rng; ++r) {
    if (v <= rng[r - 1]) {     // range r - 1 keeps at least one module
      base += steps(v);
      ++v;
    }
    const int64_t target = (n_steps * r + n_rng / 2) / n_rng;
    const int v_max = U - (n_rng - r);     // leaves a module for each later range
    while (v < v_max && base < target) {
      base += steps(v);
      ++v;
    }
    rng[r] = v;
  }
  rng[n_rng] = U;
}

}  // namespace eogp
