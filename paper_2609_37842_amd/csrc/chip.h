// The GPU's shape and the rounding helpers of the size computations (plain C++,
// no device code, so that host tests can include it).
#pragma once
#include <cstddef>
#include <cstdint>

namespace eogp {

constexpr int kXcds = 8;        // MI355X: 8 accelerator complex dies, 32 CUs each
constexpr int kCus = 256;

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
inline int64_t round_up(int64_t a, int64_t b) { return ceil_div(a, b) * b; }
inline size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

}  // namespace eogp
