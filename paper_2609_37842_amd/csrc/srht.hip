// Random second stage, EOGP-R (Appendix B.2, eq. app_srht_definition):
//   x = sqrt(p/k) R H_p D J z,  p = 2^ceil(log2 m),
// with H_p the orthonormal Walsh-Hadamard matrix. With W the unnormalised
// transform in Sylvester order (entry (r, i) = (-1)^popcount(r & i)),
//   x_c = W(D J z)[rows[c]] / sqrt(k).
//
// 1024 <= p <= 32768: one workgroup per row, E = p / NT values per thread in
// registers. The transform is separable over the bits of the index, and each
// bit's butterflies are applied once: (a) thread t loads the 16-byte pieces
// 4 t + 4 NT j of the signed, zero-padded row (one load of z and one of the
// signs per four elements) and transforms bits 0, 1 (inside a piece) and the
// bits of j in registers; (b) the values go through LDS (written 16 bytes at a
// time; a wave reads 64 consecutive words at p = 2^10, 2^12 and 2^14, two runs of 32
// at 2^11 and 2^13, and every other pair of words, half the banks, at 2^15) and
// thread t takes the elements that differ in the next log2 E bits, which are
// transformed in registers; the log2 NT - log2 E bits left are lane bits, their
// butterflies read the other lane by DPP (or permlane16_swap), not through LDS;
// (c) each thread writes its values back to the slots it read, and the kept rows
// are gathered from LDS and stored four at a time.
// What bounds it: a row's chain of phases at two rows per CU (p = 16,384; one at
// 32,768), so the instructions of each phase count. Transform and packing of 1,266
// rows, 16,384 -> 8,192: 47.5 -> 42.2 us against single-word loads and lane
// butterflies through LDS; 400 rows, 30,000 -> 8,192: 70 -> 31 us against all
// stages in LDS.
//
// p < 1024: one workgroup per row, the butterfly stages in LDS two at a time
// (radix 4: each thread combines four elements h apart), one radix-2 stage
// first when log2 p is odd. Cost either way: p log2 p additions per row, HBM
// traffic m + k floats per row.
//
// p = 65536: the same in one workgroup of 1024 threads with both halves of the
// row in registers (32 + 32 values per thread): each half is transformed as above,
// the last bit is a sum and a difference in registers, and the halves of the
// result go through LDS (128 KB) one after the other, each gathered in turn: no
// HBM traffic beyond m + k floats per row (800 rows with packing, against two
// kernels and the workspace: 50,001 -> 8,192, 410 -> 109 us; 60,000 -> 32,768,
// 588 -> 175 us).
//
// p > 65536 (up to 2^20): W_p = W_p1 (x) W_p2 in Sylvester order (index
// i = i1 p2 + i2, p2 = 32768, p1 = p / p2 <= 32). One workgroup per (row,
// chunk i1) transforms its 32768 entries along i2 as above and writes
// them to the workspace; the gather then forms each kept coordinate
// r = r1 p2 + r2 as the length-p1 transform along i1 of that column,
//   x_c = sum_j (-1)^popcount(r1 & j) S[j p2 + r2] / sqrt(k).
// Extra HBM traffic: p floats written and k p1 read per row.
#include <cmath>
#include <type_traits>

#include "common.h"
#include "timing.h"

namespace eogp {
namespace {

constexpr int kSrhtMaxLog = 15;      // a row (or half, or chunk) of 2^15 fits the LDS (128 KB)
constexpr int kSrhtMaxLogTwo = 20;   // two stages: p1 = p / 2^15 <= 32

// In-LDS unnormalised Walsh-Hadamard transform of L[0 .. 2^logp).
__device__ __forceinline__ void fwht_lds(float* L, int logp) {
  const int tid = threadIdx.x, nt = blockDim.x;
  const int p = 1 << logp;
  int h = 1;
  if (logp & 1) {                                   // one radix-2 stage (h = 1)
    for (int b = tid; b < p / 2; b += nt) {
      const float u = L[2 * b], v = L[2 * b + 1];
      L[2 * b] = u + v;
      L[2 * b + 1] = u - v;
    }
    __syncthreads();
    h = 2;
  }
  for (; h < p; h <<= 2) {                          // stages h and 2h together
    for (int b = tid; b < p / 4; b += nt) {
      // element b of the p/4 groups: low bits below h, then two group bits
      const int lo = b & (h - 1);
      const int base = ((b - lo) << 2) + lo;
      const float a0 = L[base], a1 = L[base + h], a2 = L[base + 2 * h], a3 = L[base + 3 * h];
      const float b0 = a0 + a1, b1 = a0 - a1, b2 = a2 + a3, b3 = a2 - a3;
      L[base] = b0 + b2;
      L[base + h] = b1 + b3;
      L[base + 2 * h] = b0 - b2;
      L[base + 3 * h] = b1 - b3;
    }
    __syncthreads();
  }
}

// Unnormalised Walsh-Hadamard transform of E values in registers (index j).
template <int E>
__device__ __forceinline__ void fwht_regs(float (&v)[E]) {
#pragma unroll
  for (int h = 1; h < E; h <<= 1)
#pragma unroll
    for (int j = 0; j < E; ++j)
      if ((j & h) == 0) {
        const float a = v[j], b = v[j + h];
        v[j] = a + b;
        v[j + h] = a - b;
      }
}

// Butterfly of lane bit B (B < 5): the value of lane (lane ^ 2^B) by DPP
// (quad_perm; xor 4 is a quad reversal and a half-row mirror; xor 8 a rotation
// of the row of 16), rows of 16 lanes by permlane16_swap.
template <int B>
__device__ __forceinline__ float lane_butterfly(float x, float sgn) {
  const int xi = __float_as_int(x);
  if constexpr (B == 4) {
    const auto r = __builtin_amdgcn_permlane16_swap((unsigned)xi, (unsigned)xi, false, false);
    return fmaf(sgn, __uint_as_float(r[1]), __uint_as_float(r[0]));   // even row +- odd row
  } else {
    int o;
    if constexpr (B == 0)
      o = __builtin_amdgcn_mov_dpp(xi, 0xB1, 0xF, 0xF, false);        // quad_perm 1 0 3 2
    else if constexpr (B == 1)
      o = __builtin_amdgcn_mov_dpp(xi, 0x4E, 0xF, 0xF, false);        // quad_perm 2 3 0 1
    else if constexpr (B == 2)
      o = __builtin_amdgcn_mov_dpp(__builtin_amdgcn_mov_dpp(xi, 0x1B, 0xF, 0xF, false), 0x141, 0xF,
                                   0xF, false);                        // ^3, then ^7
    else
      o = __builtin_amdgcn_mov_dpp(xi, 0x128, 0xF, 0xF, false);       // row_ror:8
    return fmaf(sgn, x, __int_as_float(o));   // sgn is 1 or -1: exactly o + x or o - x
  }
}

typedef float f4_any __attribute__((ext_vector_type(4), aligned(4)));     // at any element
typedef int i4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32_any __attribute__((aligned(1)));                     // four signs

// 2^LOGP elements by 2^LT threads, E per thread.
template <int LOGP, int LT>
struct RowFwht {
  static constexpr int NT = 1 << LT, P = 1 << LOGP, LE = LOGP - LT, E = 1 << LE, LB = LT - LE;
  static_assert(LE >= 2 && LB >= 0 && LB <= 5, "the lane bits of phase (b) lie below bit 5");

  // (a) pieces 4 t + 4 NT j of the row's first `have` elements (have <= P, the
  // rest zero). The loads are at clamped places, so that all are in flight at
  // once; the one piece that `have` cuts is loaded again element by element.
  static __device__ __forceinline__ void load(float (&v)[E], const float* __restrict__ z,
                                              const int8_t* __restrict__ signs, int have, int t) {
    f4_any zq[E / 4];
    uint32_t sg[E / 4];
    if (have >= 4) {
#pragma unroll
      for (int j = 0; j < E / 4; ++j) {
        const int at = min(4 * t + 4 * NT * j, have - 4);
        zq[j] = *reinterpret_cast<const f4_any*>(z + at);
        sg[j] = *reinterpret_cast<const u32_any*>(signs + at);
      }
    }
#pragma unroll
    for (int j = 0; j < E / 4; ++j) {
      const int at = 4 * t + 4 * NT * j;
      if (at + 4 > have) {                     // cut by the row's end, or past it
        zq[j] = f4_any{0.f, 0.f, 0.f, 0.f};
        sg[j] = 0;
        for (int c = 0; c < 3; ++c)
          if (at + c < have) {
            zq[j][c] = z[at + c];
            sg[j] |= (uint32_t)(uint8_t)signs[at + c] << (8 * c);
          }
      }
#pragma unroll
      for (int c = 0; c < 4; ++c)
        v[4 * j + c] = __uint_as_float(__float_as_uint(zq[j][c]) ^ ((sg[j] << (24 - 8 * c)) & 0x80000000u));
    }
  }

  // Place of value e of thread t after transform(): thread bits 0 .. LB - 1 are
  // index bits 2 .., e the LE bits above them, thread bits LB, LB + 1 index bits
  // 0 and 1, the rest the top ones.
  static __device__ __forceinline__ int place(int t, int e) {
    return ((t & ((1 << LB) - 1)) << 2) | ((t >> LB) & 3) | ((t >> (LB + 2)) << (LT + 2)) | (e << (2 + LB));
  }

  // In: v as load() leaves it; out: the transform, value e at place(t, e). L's
  // former content is no longer read when a thread enters; when the call returns,
  // a thread may overwrite its own places only, until the next barrier.
  static __device__ __forceinline__ void transform(float (&v)[E], float* L, int t) {
    fwht_regs<E>(v);
#pragma unroll
    for (int j = 0; j < E / 4; ++j)
      *reinterpret_cast<float4*>(L + 4 * t + 4 * NT * j) =
          make_float4(v[4 * j], v[4 * j + 1], v[4 * j + 2], v[4 * j + 3]);
    __syncthreads();
#pragma unroll
    for (int e = 0; e < E; ++e) v[e] = L[place(t, e)];
    fwht_regs<E>(v);
    auto cross = [&](auto b_c) __attribute__((always_inline)) {
      constexpr int B = decltype(b_c)::value;
      const float sgn = (t >> B) & 1 ? -1.f : 1.f;
#pragma unroll
      for (int e = 0; e < E; ++e) v[e] = lane_butterfly<B>(v[e], sgn);
    };
    if constexpr (LB > 0) cross(std::integral_constant<int, 0>{});
    if constexpr (LB > 1) cross(std::integral_constant<int, 1>{});
    if constexpr (LB > 2) cross(std::integral_constant<int, 2>{});
    if constexpr (LB > 3) cross(std::integral_constant<int, 3>{});
    if constexpr (LB > 4) cross(std::integral_constant<int, 4>{});
  }

  static __device__ __forceinline__ void put(const float (&v)[E], float* L, int t) {
#pragma unroll
    for (int e = 0; e < E; ++e) L[place(t, e)] = v[e];
  }
};

template <int LOGP, int LT>
__global__ __launch_bounds__(1 << LT) void k_srht_reg(const float* __restrict__ Z, int64_t ldz, int m,
                                                      const int8_t* __restrict__ signs,
                                                      const int32_t* __restrict__ rows, int k,
                                                      float scale, float* __restrict__ X, int64_t ldx) {
  using R = RowFwht<LOGP, LT>;
  extern __shared__ float4 L4[];
  float* L = reinterpret_cast<float*>(L4);
  const int t = threadIdx.x;
  const int64_t i = blockIdx.x;
  float v[R::E];
  R::load(v, Z + i * ldz, signs, m, t);
  R::transform(v, L, t);
  R::put(v, L, t);
  __syncthreads();
  // (c) gather (k <= p, so at most E / 4 pieces of four per thread): every
  // index requested before the first is used
  float* x = X + i * ldx;
  auto kept = [&](int r) __attribute__((always_inline)) {
    return (unsigned)r < (unsigned)R::P ? L[r] * scale : __builtin_nanf("");
  };
  i4_any r[R::E / 4];
#pragma unroll
  for (int q = 0; q < R::E / 4; ++q) {
    const int c = 4 * t + 4 * R::NT * q;
    if (c + 4 <= k) r[q] = *reinterpret_cast<const i4_any*>(rows + c);
  }
#pragma unroll
  for (int q = 0; q < R::E / 4; ++q) {
    const int c = 4 * t + 4 * R::NT * q;
    if (c + 4 <= k)
      *reinterpret_cast<f4_any*>(x + c) = f4_any{kept(r[q].x), kept(r[q].y), kept(r[q].z), kept(r[q].w)};
    else
      for (int u = 0; u < 3; ++u)
        if (c + u < k) x[c + u] = kept(rows[c + u]);
  }
}

// p = 65536: the halves of the row in v and w, their sum and difference (index
// bit 15) in registers, each gathered from LDS in its turn.
__global__ __launch_bounds__(1024) void k_srht_two(const float* __restrict__ Z, int64_t ldz, int m,
                                                   const int8_t* __restrict__ signs,
                                                   const int32_t* __restrict__ rows, int k,
                                                   float scale, float* __restrict__ X, int64_t ldx) {
  using R = RowFwht<kSrhtMaxLog, 10>;
  extern __shared__ float4 L4[];
  float* L = reinterpret_cast<float*>(L4);
  const int t = threadIdx.x;
  const int64_t i = blockIdx.x;
  const float* z = Z + i * ldz;
  float v[R::E], w[R::E];
  R::load(v, z, signs, R::P, t);
  R::load(w, z + R::P, signs + R::P, m - R::P, t);
  R::transform(v, L, t);
  __syncthreads();                                  // every read of the first half is done
  R::transform(w, L, t);
#pragma unroll
  for (int e = 0; e < R::E; ++e) {
    const float a = v[e], b = w[e];
    v[e] = a + b;
    w[e] = a - b;
  }
  float* x = X + i * ldx;
  // the kept rows among first .. first + R::P - 1 (and, the first time, the bad
  // ones); eight indices requested before the first is used
  auto gather = [&](int first) __attribute__((always_inline)) {
    for (int c0 = t; c0 < k; c0 += 8 * R::NT) {
      int r[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) r[u] = rows[min(c0 + R::NT * u, k - 1)];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int c = c0 + R::NT * u;
        if (c < k && (unsigned)r[u] - (unsigned)first < (unsigned)R::P) x[c] = L[r[u] - first] * scale;
        else if (c < k && first == 0 && (unsigned)r[u] >= 2u * R::P) x[c] = __builtin_nanf("");
      }
    }
  };
  R::put(v, L, t);
  __syncthreads();
  gather(0);
  __syncthreads();
  R::put(w, L, t);
  __syncthreads();
  gather(R::P);
}

__global__ __launch_bounds__(1024) void k_srht(const float* __restrict__ Z, int64_t ldz, int m,
                                               int logp, const int8_t* __restrict__ signs,
                                               const int32_t* __restrict__ rows, int k,
                                               float scale, float* __restrict__ X, int64_t ldx) {
  extern __shared__ float L[];
  const int64_t i = blockIdx.x;
  const int tid = threadIdx.x, nt = blockDim.x;
  const int p = 1 << logp;
  const float* z = Z + i * ldz;
  for (int c = tid; c < p; c += nt) {
    float v = 0.f;
    if (c < m) v = signs[c] < 0 ? -z[c] : z[c];
    L[c] = v;
  }
  __syncthreads();
  fwht_lds(L, logp);
  float* x = X + i * ldx;
  for (int c = tid; c < k; c += nt) {
    const int r = rows[c];
    x[c] = (r >= 0 && r < p) ? L[r] * scale : __builtin_nanf("");
  }
}

// Two-stage form, first stage: grid (p1, N); chunk i1 of row i, signed and
// zero-padded, transformed along i2 into S[i][i1 p2 ..].
__global__ __launch_bounds__(1024) void k_srht_chunk(const float* __restrict__ Z, int64_t ldz,
                                                     int m, const int8_t* __restrict__ signs,
                                                     float* __restrict__ S, int64_t lds_row) {
  using R = RowFwht<kSrhtMaxLog, 10>;
  extern __shared__ float4 L4[];
  const int t = threadIdx.x;
  const int64_t i = blockIdx.y;
  const int c0 = (int)blockIdx.x << kSrhtMaxLog;
  const int have = min(max(m - c0, 0), R::P);
  float v[R::E];
  R::load(v, Z + i * ldz + (have ? c0 : 0), signs + (have ? c0 : 0), have, t);
  R::transform(v, reinterpret_cast<float*>(L4), t);
  float* out = S + i * lds_row + c0;
#pragma unroll
  for (int e = 0; e < R::E; ++e) out[R::place(t, e)] = v[e];
}

// Second stage fused with the gather: grid (ceil(k / 256), N).
__global__ __launch_bounds__(256) void k_srht_cross(const float* __restrict__ S, int64_t lds_row,
                                                    int logp, const int32_t* __restrict__ rows,
                                                    int k, float scale, float* __restrict__ X,
                                                    int64_t ldx) {
  const int64_t i = blockIdx.y;
  const int c = blockIdx.x * 256 + threadIdx.x;
  if (c >= k) return;
  const int p = 1 << logp, p1 = 1 << (logp - kSrhtMaxLog);
  const int r = rows[c];
  if (r < 0 || r >= p) {
    X[i * ldx + c] = __builtin_nanf("");
    return;
  }
  const int r1 = r >> kSrhtMaxLog, r2 = r & ((1 << kSrhtMaxLog) - 1);
  const float* col = S + i * lds_row + r2;
  float acc = 0.f;
  for (int j = 0; j < p1; ++j) {
    const float v = col[(int64_t)j << kSrhtMaxLog];
    acc += (__popc(r1 & j) & 1) ? -v : v;
  }
  X[i * ldx + c] = acc * scale;
}

}  // namespace

int srht_max_log() { return kSrhtMaxLogTwo; }

namespace {
int srht_log(int64_t m) {
  int logp = 0;
  while ((int64_t(1) << logp) < m) ++logp;
  return logp;
}
}  // namespace

size_t srht_ws(int64_t N, int64_t m) {
  const int logp = srht_log(m);
  if (logp <= kSrhtMaxLog) return 0;
  return align256((size_t)N * ((size_t)1 << logp) * sizeof(float));
}

eogp_status srht_project(const float* Z, int64_t ldz, int64_t N, int64_t m, const int8_t* signs,
                         const int32_t* rows, int64_t k, float* X, int64_t ldx, void* ws,
                         size_t ws_bytes, hipStream_t s) {
  if (N == 0) return EOGP_OK;
  const int logp = srht_log(m);
  const float scale = (float)(1.0 / std::sqrt((double)k));
  if (logp < 10) {
    timing::Scope ts(EOGP_KT_SRHT, s);
    const int p = 1 << logp;
    const size_t lds = (size_t)p * sizeof(float);
    const int nt = std::max(64, std::min(1024, p / 4));
    for (int64_t r0 = 0; r0 < N; r0 += 0x7FFFFFFF) {
      const int64_t nr = std::min<int64_t>(N - r0, 0x7FFFFFFF);
      hipLaunchKernelGGL(k_srht, dim3((unsigned)nr), dim3(nt), lds, s, Z + r0 * ldz, ldz, (int)m,
                         logp, signs, rows, (int)k, scale, X + r0 * ldx, ldx);
      EOGP_LAUNCH_CHECK("srht_project");
    }
    return EOGP_OK;
  }
  if (logp <= kSrhtMaxLog + 1) {
    // One row per workgroup. The two-half kernel needs no workspace; a call of
    // its size still has to bring the one that srht_ws states, as it always had to.
    if (logp > kSrhtMaxLog && (ws_bytes < srht_ws(N, m) || !ws))
      return fail(EOGP_ERR_WORKSPACE, "srht_project: workspace too small");
    using Kernel = void (*)(const float*, int64_t, int, const int8_t*, const int32_t*, int, float,
                            float*, int64_t);
    static constexpr Kernel fns[7] = {k_srht_reg<10, 7>, k_srht_reg<11, 7>, k_srht_reg<12, 8>,
                                      k_srht_reg<13, 8>, k_srht_reg<14, 9>, k_srht_reg<15, 10>, k_srht_two};
    static constexpr int lts[7] = {7, 7, 8, 8, 9, 10, 10};
    const Kernel fn = fns[logp - 10];
    const int lds = (int)(sizeof(float) << std::min(logp, kSrhtMaxLog));
    const eogp_status st = ensure_dynamic_lds((const void*)fn, lds);
    if (st != EOGP_OK) return st;
    timing::Scope ts(EOGP_KT_SRHT, s);
    for (int64_t r0 = 0; r0 < N; r0 += 0x7FFFFFFF) {
      const int64_t nr = std::min<int64_t>(N - r0, 0x7FFFFFFF);
      hipLaunchKernelGGL(fn, dim3((unsigned)nr), dim3(1u << lts[logp - 10]), lds, s, Z + r0 * ldz, ldz,
                         (int)m, signs, rows, (int)k, scale, X + r0 * ldx, ldx);
      EOGP_LAUNCH_CHECK("srht_project");
    }
    return EOGP_OK;
  }
  if (ws_bytes < srht_ws(N, m) || !ws) return fail(EOGP_ERR_WORKSPACE, "srht_project: workspace too small");
  const eogp_status st = ensure_dynamic_lds((const void*)k_srht_chunk, (int)(sizeof(float) << kSrhtMaxLog));
  if (st != EOGP_OK) return st;
  timing::Scope ts(EOGP_KT_SRHT, s);
  float* S = static_cast<float*>(ws);
  const int64_t p = int64_t(1) << logp;
  const int p1 = 1 << (logp - kSrhtMaxLog);
  for (int64_t r0 = 0; r0 < N; r0 += 65535) {
    const int64_t nr = std::min<int64_t>(N - r0, 65535);
    hipLaunchKernelGGL(k_srht_chunk, dim3((unsigned)p1, (unsigned)nr), dim3(1024),
                       sizeof(float) << kSrhtMaxLog, s, Z + r0 * ldz, ldz, (int)m, signs,
                       S + r0 * p, p);
    hipLaunchKernelGGL(k_srht_cross, dim3((unsigned)ceil_div(k, 256), (unsigned)nr), dim3(256), 0,
                       s, S + r0 * p, p, logp, rows, (int)k, scale, X + r0 * ldx, ldx);
    EOGP_LAUNCH_CHECK("srht_project (two stages)");
  }
  return EOGP_OK;
}

}  // namespace eogp
