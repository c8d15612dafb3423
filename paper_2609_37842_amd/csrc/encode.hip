// Second stage (eq. second_stage) and one-bit encoding (eq. onebit).
#include <algorithm>

#include "gemm.h"
#include "timing.h"

namespace eogp {
namespace {

// One workgroup (4 waves) per row, HBM-bound. Wave w takes the 256-coordinate
// chunks w, w + 4, ...; each lane loads four consecutive coordinates (16 bytes, at
// any element) of UNR chunks before it uses the first: eight, so a row of up to
// 8,192 coordinates is in flight at once; as few as hold a shorter row, because every
// chunk past its end still costs its bounds checks (20,000 rows of 64: 32.9 us with
// eight chunks, 14.9 with one). A lane's four signs are a nibble; eight lanes
// combine theirs by DPP into four bytes of the least-significant-bit-first code
// (coordinate 4 l + c of a chunk is bit c of lane l's nibble). |x| is summed in
// fp64 (per lane, then a fixed butterfly, then the four waves in order) and the
// mean is rounded once to fp16.
// 1,266 rows of 8,192 into a tiled store: 11.7 -> 9.8 us against one word per lane
// and a ballot per 64 coordinates; 400 rows transformed and packed: 31.3 -> 28.9 us.
//
// Tiled store (TILED): rows in tiles of 32; the 64 bytes of row r in 512-bit
// step s of the row (a module's steps start at step0) go to the 2 KB block
// (tile * steps_row + s), 16-byte piece p (bytes 16p .. 16p+15) at block
// offset (p % 2) * 1024 + ((p / 2) * 32 + r) * 16: the order in which the
// scoring pass's wave lanes take them (k a multiple of 512).
typedef float f4_any __attribute__((ext_vector_type(4), aligned(4)));

// OR over the eight lanes 8 i .. 8 i + 7, in every one of them.
__device__ __forceinline__ uint32_t or_lanes8(uint32_t x) {
  x |= (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0xB1, 0xF, 0xF, false);    // lane ^ 1
  x |= (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x4E, 0xF, 0xF, false);    // lane ^ 2
  x |= (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x141, 0xF, 0xF, false);   // half-row mirror: the other quad
  return x;
}

template <bool TILED, int UNR>
__global__ __launch_bounds__(256) void k_sign_pack(const float* __restrict__ X, int64_t ldx,
                                                   int64_t N, int64_t k,
                                                   uint8_t* __restrict__ codes, int64_t cstride,
                                                   uint16_t* __restrict__ scales,
                                                   int64_t sstride, int word_store, int64_t row0,
                                                   int64_t steps_row, int64_t step0) {
  __shared__ double part[4];
  const int64_t i = blockIdx.x;
  const int wid = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const float* x = X + i * ldx;
  uint8_t* c = codes + i * cstride;
  const int64_t grow = row0 + i;   // tiled: the row's place in the store
  uint8_t* tb = codes + ((grow >> 5) * steps_row + step0) * 2048 + (grow & 31) * 16;
  const int64_t nchunk = (k + 255) >> 8, nbytes = (k + 7) >> 3;
  double acc = 0.0;
  for (int64_t ch0 = wid; ch0 < nchunk; ch0 += 4 * UNR) {
    f4_any v[UNR];
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      const int64_t c0 = (ch0 + 4 * u) * 256 + 4 * lane;
      if (TILED || c0 + 4 <= k) {
        if (c0 < k) v[u] = *reinterpret_cast<const f4_any*>(x + c0);
      } else {
        v[u] = f4_any{0.f, 0.f, 0.f, 0.f};         // the row's end, and past it
        for (int e = 0; e < 3; ++e)
          if (c0 + e < k) v[u][e] = x[c0 + e];
      }
    }
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      const int64_t ch = ch0 + 4 * u;
      if (ch >= nchunk) break;                     // uniform across the wave
      const int64_t c0 = ch * 256 + 4 * lane;
      uint32_t nib = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (TILED || c0 + e < k) nib |= (v[u][e] >= 0.f ? 1u : 0u) << e;
        acc += fabs((double)v[u][e]);              // 0 beyond k
      }
      const uint32_t word = or_lanes8(nib << (4 * (lane & 7)));
      if ((lane & 7) == 0) {
        const int d = lane >> 3;                   // bytes 4 d .. 4 d + 3 of the chunk's 32
        if constexpr (TILED) {
          // step ch / 2; its pieces 2 (ch % 2) + d / 4
          *reinterpret_cast<uint32_t*>(tb + (ch >> 1) * 2048 + (d >> 2) * 1024 + (ch & 1) * 512 +
                                       (d & 3) * 4) = word;
        } else {
          const int64_t at = ch * 32 + 4 * d;
          if (word_store && at + 4 <= nbytes) {
            *reinterpret_cast<uint32_t*>(c + at) = word;
          } else {
            for (int b = 0; b < 4; ++b)
              if (at + b < nbytes) c[at + b] = (uint8_t)(word >> (8 * b));
          }
        }
      }
    }
  }
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
  if (lane == 0) part[wid] = acc;
  __syncthreads();
  if (threadIdx.x == 0)
    scales[i * sstride] = f64_to_f16_rne(((part[0] + part[1]) + (part[2] + part[3])) / (double)k);
}

// fp32 P (column-major, [k][ldp]) -> bf16 high and low parts [k][ldo].
__global__ void k_split_p(const float* __restrict__ P, int64_t ldp, int64_t m, int64_t k,
                          int64_t ldo, uint16_t* __restrict__ hi, uint16_t* __restrict__ lo) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t col = idx / ldo, r = idx % ldo;
  const float v = (r < m && col < k) ? P[col * ldp + r] : 0.f;   // zero padding
  const uint16_t h = to_bf16_bits(v);
  hi[idx] = h;
  lo[idx] = to_bf16_bits(v - bf16_bits_to_f32(h));
}

template <bool TILED>
void launch_pack(const float* X, int64_t ldx, int64_t N, int64_t k, uint8_t* codes, int64_t cstride,
                 uint16_t* scales, int64_t sstride, int word_store, int64_t row0, int64_t steps_row,
                 int64_t step0, hipStream_t s) {
  auto* kfn = k <= 1024   ? k_sign_pack<TILED, 1>
              : k <= 2048 ? k_sign_pack<TILED, 2>
              : k <= 4096 ? k_sign_pack<TILED, 4>
                          : k_sign_pack<TILED, 8>;
  hipLaunchKernelGGL(kfn, dim3((unsigned)N), dim3(256), 0, s, X, ldx, N, k, codes, cstride, scales,
                     sstride, word_store, row0, steps_row, step0);
}

}  // namespace

eogp_status sign_pack(const float* X, int64_t ldx, int64_t N, int64_t k, uint8_t* codes,
                      int64_t cstride, uint16_t* scales, int64_t sstride, hipStream_t s) {
  if (N == 0) return EOGP_OK;
  const int word_store = ((uintptr_t)codes % 4 == 0) && (cstride % 4 == 0);
  timing::Scope ts(EOGP_KT_SIGN_PACK, s);
  launch_pack<false>(X, ldx, N, k, codes, cstride, scales, sstride, word_store, 0, 0, 0, s);
  EOGP_LAUNCH_CHECK("sign_pack");
  return EOGP_OK;
}

eogp_status sign_pack_tiled(const float* X, int64_t ldx, int64_t N, int64_t k, int64_t row0,
                            uint8_t* codes, int64_t steps_row, int64_t step0, uint16_t* scales,
                            int64_t sstride, hipStream_t s) {
  if (N == 0) return EOGP_OK;
  timing::Scope ts(EOGP_KT_SIGN_PACK, s);
  launch_pack<true>(X, ldx, N, k, codes, 0, scales, sstride, 0, row0, steps_row, step0, s);
  EOGP_LAUNCH_CHECK("sign_pack (tiled)");
  return EOGP_OK;
}

constexpr int kPcaMaxSplits = 8;

// Workspace: the split copy of an fp32 P (padded panel), then split-K partials.
size_t pca_split_copy_bytes(int64_t m, int64_t k, eogp_dtype p_dtype) {
  if (p_dtype != EOGP_F32) return 0;
  const int64_t ldo = round_up(m, 32), rows = round_up(k, 256);
  return 2 * align256((size_t)rows * ldo * 2);
}

size_t pca_ws(int64_t N, int64_t m, int64_t k, eogp_dtype p_dtype) {
  return pca_split_copy_bytes(m, k, p_dtype) +
         align256(gemm_partial_bytes(N, k, kPcaMaxSplits));
}

eogp_status pca_project(const void* Z, eogp_dtype z_dtype, int64_t ldz, int64_t N, int64_t m,
                        const void* P, eogp_dtype p_dtype, int64_t ldp, int64_t k, float* X,
                        int64_t ldx, bool accurate, void* ws, size_t ws_bytes, hipStream_t s) {
  if (N == 0 || k == 0) return EOGP_OK;
  GemmArgs g;
  g.A = Z;
  g.lda = ldz;
  g.C = X;
  g.ldc = ldx;
  g.M = N;
  g.N = k;
  g.K = m;
  // Units run split by split (each XCD's contiguous range is then one K
  // range), column tile by column tile with the row tiles of a column tile
  // together: each P slice is fetched once and shared by the row tiles, and
  // the Z slices of the K range stay in that XCD's L2.
  g.n_major = true;
  g.split_major = true;
  g.timing_class = EOGP_KT_PCA_GEMM;
  const size_t copy = pca_split_copy_bytes(m, k, p_dtype);
  if (ws_bytes < copy) return fail(EOGP_ERR_WORKSPACE, "pca_project: workspace too small");
  // Split-K scratch is optional: without it the projection runs unsplit.
  if (ws && ws_bytes >= copy + gemm_partial_bytes(N, k, 2)) {
    g.partial = reinterpret_cast<float*>(static_cast<char*>(ws) + copy);
    g.max_splits = (int)std::min<int64_t>(
        kPcaMaxSplits, (int64_t)((ws_bytes - copy) / gemm_partial_bytes(N, k, 1)));
  }
  if (p_dtype == EOGP_F32) {   // (Z is fp32 here)
    const int64_t ldo = round_up(m, 32), rows = round_up(k, 256);
    Carve cv(ws, ws_bytes);
    uint16_t* hi = cv.take<uint16_t>((size_t)rows * ldo);
    uint16_t* lo = cv.take<uint16_t>((size_t)rows * ldo);
    const int64_t total = rows * ldo;
    hipLaunchKernelGGL(k_split_p, dim3((unsigned)ceil_div(total, 256)), dim3(256), 0, s,
                       static_cast<const float*>(P), ldp, m, k, ldo, hi, lo);
    EOGP_LAUNCH_CHECK("pca split");
    g.B_hi = hi;
    g.B_lo = lo;
    g.ldb = ldo;
    g.b_padded = true;
    return gemm_nt(g, AType::F32, accurate ? 2 : 1, accurate ? 2 : 1, false, s);
  }
  g.B_hi = static_cast<const uint16_t*>(P);
  g.ldb = ldp;
  // 16-bit Z has P's type (checked by the caller): one product on that type's MFMA
  if (z_dtype != EOGP_F32) return gemm_nt(g, AType::B16, 1, 1, p_dtype == EOGP_F16, s);
  return gemm_nt(g, AType::F32, accurate ? 2 : 1, 1, p_dtype == EOGP_F16, s);
}

}  // namespace eogp
