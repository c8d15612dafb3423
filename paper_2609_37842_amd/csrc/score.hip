// Scoring stored one-bit codes against unquantized query projections
// (eq. onebit_influence, eq. app_stored_influence) with a per-query top-k.
//
// Arithmetic. Each query module vector y is taken in fixed point,
// y_int = rint(y 2^f) with f = 14 - e for max|y| = mu 2^e (|y_int| <= 2^14), and
// split into two int8 planes y_int = 256 h + l (h in [-64, 64], l in
// [-128, 127]). With b in {0, 1} the MFMAs compute n1 = sum_{b=1} y_int exactly
// in integers, and <y_int, 2b - 1> = 2 n1 - sum(y_int). Each module term
// s * (2 n1 - sum) * 2^-f is exact in fp64 and the terms are added in module
// order, so the score is reproducible bit for bit.
//
// Data flow. A pass streams every stored code once for a group of NQT * 16
// queries (NQT = 2: 32, the rule is in choose_cfg). v_mfma_i32_32x32x32_i8
// takes the 32 plane rows of 16 queries ({h, l}) as its A operand and 32
// stored rows as B, so one instruction serves both planes and each lane ends
// with 8 queries of one stored row (the h and l sums of a query land in the
// same lane). A 512-thread workgroup (8 waves, 2 per SIMD) owns 256 RT
// consecutive rows at a time, each wave RT tiles of 32 rows. The modules are
// walked in steps of 512 bits, each in two halves of 256: per half each lane
// holds 16 bytes of each of its RT rows (requested again as soon as they are used,
// or, for row-major rows a multiple of 8 KB apart, both halves together a step
// ahead), the workgroup stages the half's plane fragments (8 KB per 16 queries) in
// LDS, and every fragment read from LDS feeds RT MFMAs, every expanded code operand
// NQT of them. The requests run on into the next block of rows, so a block's
// last halves and its candidate pass cover the next one's first loads.
//
// Bit expansion. The 16 bytes c of a lane feed 8 MFMAs per query tile, one per
// bit position t of a byte. The operand of MFMA t is (c >> s) & (0x01010101 <<
// w) with t = s + w, w = t mod NCLS: its bytes are 0 or 2^w, so the MFMA adds
// 2^w times the wanted sum into accumulator class w, and n1 = sum_w acc_w /
// 2^w (exact shifts: every term of acc_w is a multiple of 2^w). One 64-bit
// shift serves two words, and with NCLS = 2 one shift serves two masks: 32 ANDs
// and 6 shifts for 16 bytes; NCLS = 1 (NQT = 2, whose accumulators take the
// registers of the second class) takes 32 ANDs and 14 shifts for twice as
// many MFMAs. The query planes are prepared in exactly that order: byte j of
// lane (M, g) of MFMA (u, t) in step s of a module holds coordinate 8 (64 s +
// o + j) + t, where o = 32 g + 16 u for the tiled store (its 16-byte pieces)
// and 32 u + 16 g for row-major rows (each half then reads 32 bytes of a row
// together).
//
// After the last module the workgroup's scores are filtered against a
// per-query threshold into an LDS candidate list (score desc, index asc). The
// threshold starts at the top-k-th largest of the first block's per-lane
// maxima (that many rows reach it, so no row below it can be kept). A list
// that fills up is pruned to its top-k by one wave (a bitwise search of the
// k-th key over ballots, eight lists at a time) and the entries that did not
// fit are offered again, so no qualifying row is lost. Finally each workgroup
// writes its top-k per query and a merge kernel reduces them.
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "common.h"
#include "score_plan.h"
#include "timing.h"

namespace eogp {
namespace {

constexpr int NTHR = NW * 64;
constexpr int MAX_TOPK = 256;
constexpr int HALF_U4 = 8 * 64;        // 16-byte slots of a half step's fragments per 16 queries

typedef __attribute__((__vector_size__(16 * sizeof(int)))) int i32x16;
template <typename T>
using cptr = const __attribute__((address_space(4))) T*;   // read-only, scalar loads

// A shift amount the compiler does not know: a 64-bit shift by it stays one
// instruction. (Of a shift by a known amount whose crossing bits are masked away
// the compiler makes two 32-bit ones.)
__device__ __forceinline__ int opaque_shift(int s) {
  asm("" : "+s"(s));
  return s;
}

__device__ __forceinline__ uint64_t order_key(double x) {
  uint64_t u = (uint64_t)__double_as_longlong(x);
  return (u >> 63) ? ~u : (u | 0x8000000000000000ull);
}
__device__ __forceinline__ double key_value(uint64_t k) {
  uint64_t u = (k >> 63) ? (k & 0x7FFFFFFFFFFFFFFFull) : ~k;
  return __longlong_as_double((long long)u);
}
__device__ __forceinline__ bool before(uint64_t ka, uint32_t ia, uint64_t kb, uint32_t ib) {
  return ka > kb || (ka == kb && ia < ib);
}

// ---- query preparation --------------------------------------------------------
// grid (16 * groups, U): per (query, module) the exponent f and the sum of
// y_int, stored [group][U][16]; queries past Q get f = 0 and sum 0. The sum is
// carried in 64 bits: |y_int| <= 2^14 and k_u <= 2^22 bound it by 2^36.
// One 512-thread workgroup, eight loads in flight per thread: with 256 threads
// and one load at a time the chain of loads was the whole time (16 queries of
// 16,384 coordinates 40 us; now 11 us).
constexpr int STAT_THR = 512, STAT_UNR = 8;
__global__ __launch_bounds__(STAT_THR) void k_query_stats(const float* __restrict__ Y, int64_t ldy,
                                                          int64_t Q, int U,
                                                          const ModInfo* __restrict__ mods,
                                                          int32_t* __restrict__ fq,
                                                          int64_t* __restrict__ ysum) {
  __shared__ float smax[STAT_THR / 64];
  __shared__ int64_t ssum[STAT_THR / 64];
  const int64_t q = blockIdx.x;
  const int u = blockIdx.y, tid = threadIdx.x;
  const int64_t o = ((q / QB) * U + u) * QB + (q % QB);
  if (q >= Q) {
    if (tid == 0) {
      fq[o] = 0;
      ysum[o] = 0;
    }
    return;
  }
  const ModInfo md = mods[u];
  const float* y = Y + q * ldy + md.coff;
  float mx = 0.f;
  for (int c = tid; c < md.k; c += STAT_THR * STAT_UNR) {
    float v[STAT_UNR];
#pragma unroll
    for (int e = 0; e < STAT_UNR; ++e) v[e] = y[min(c + e * STAT_THR, md.k - 1)];
#pragma unroll
    for (int e = 0; e < STAT_UNR; ++e) mx = fmaxf(mx, fabsf(v[e]));
  }
  for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
  if ((tid & 63) == 0) smax[tid >> 6] = mx;
  __syncthreads();
  mx = smax[0];
#pragma unroll
  for (int w = 1; w < STAT_THR / 64; ++w) mx = fmaxf(mx, smax[w]);
  int f = 0;
  if (mx > 0.f) {
    int e;
    (void)frexpf(mx, &e);
    f = 14 - e;
  }
  int64_t s = 0;
  if (mx > 0.f)
    for (int c = tid; c < md.k; c += STAT_THR * STAT_UNR) {
      float v[STAT_UNR];
#pragma unroll
      for (int e = 0; e < STAT_UNR; ++e) v[e] = y[min(c + e * STAT_THR, md.k - 1)];
#pragma unroll
      for (int e = 0; e < STAT_UNR; ++e)
        if (c + e * STAT_THR < md.k) s += (int64_t)rintf(ldexpf(v[e], f));
    }
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
  if ((tid & 63) == 0) ssum[tid >> 6] = s;
  __syncthreads();
  if (tid == 0) {
    fq[o] = f;
    int64_t t = 0;
    for (int w = 0; w < STAT_THR / 64; ++w) t += ssum[w];
    ysum[o] = t;
  }
}

// Writes entries first .. first + count - 1 of the module table. The table
// travels in the kernel arguments (copied when the launch is enqueued), so
// the call needs no host synchronisation and the host's copy may go at once.
constexpr int MOD_CHUNK = 64;
struct ModChunk {
  ModInfo m[MOD_CHUNK];
  int32_t first, count;
};
__global__ void k_mod_table(ModChunk c, ModInfo* __restrict__ mods) {
  const int i = threadIdx.x;
  if (i < c.count) mods[c.first + i] = c.m[i];
}

// Planes laid out [group][step][MFMA f][lane][j] with f = 8 u + t: lane
// (M, g) = (lane % 32, lane / 32) is plane M / 16 (0: h, 1: l) of query M % 16,
// byte j holds coordinate 8 (64 s + o + j) + t of the step's module (0 past the
// module), o = 32 g + 16 u (tiled) or 32 u + 16 g. One thread per (group, step,
// u, g, query, t) forms the 16 bytes of both planes of its query: eight
// neighbouring threads (t = 0..7) read eight neighbouring coordinates.
__global__ __launch_bounds__(256) void k_query_planes(const float* __restrict__ Y, int64_t ldy,
                                                      int64_t Q, int U,
                                                      const ModInfo* __restrict__ mods,
                                                      const int32_t* __restrict__ fq,
                                                      int64_t n_steps, int64_t n_groups, int tiled,
                                                      int8_t* __restrict__ planes) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= n_groups * n_steps * 512) return;
  const int t = (int)(idx & 7);
  const int qn = (int)((idx >> 3) & 15);
  const int g = (int)((idx >> 7) & 1);
  const int uc = (int)((idx >> 8) & 1);
  const int64_t gs = idx >> 9;
  const int64_t step = gs % n_steps;
  const int64_t grp = gs / n_steps;
  int lo = 0, hi = U - 1;                    // last module whose first step <= step
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (mods[mid].sbase <= step) lo = mid; else hi = mid - 1;
  }
  const ModInfo md = mods[lo];
  const int64_t sl = step - md.sbase;
  const int64_t q = grp * QB + qn;
  const int f = q < Q ? fq[(grp * U + lo) * QB + qn] : 0;
  const int o = tiled ? 32 * g + 16 * uc : 32 * uc + 16 * g;
  const int64_t c0 = 8 * (SB * sl + o) + t;                 // coordinate of byte 0
  const float* y = Y + q * ldy + md.coff;
  uint32_t hw[4] = {0u, 0u, 0u, 0u}, lw[4] = {0u, 0u, 0u, 0u};
#pragma unroll
  for (int jj = 0; jj < 16; ++jj) {
    const int64_t c = c0 + 8 * jj;
    int yi = 0;
    if (q < Q && c < md.k) yi = (int)rintf(ldexpf(y[c], f));
    const int h = (yi + 128) >> 8;   // floor division (arithmetic shift)
    const int l = yi - 256 * h;
    hw[jj >> 2] |= (uint32_t)(h & 0xFF) << (8 * (jj & 3));
    lw[jj >> 2] |= (uint32_t)(l & 0xFF) << (8 * (jj & 3));
  }
  int8_t* blk = planes + (gs * FRAGS + 8 * uc + t) * 1024;
  const int lane = qn + 32 * g;   // plane h; plane l is lane + 16
  *reinterpret_cast<uint4*>(blk + 16 * lane) = make_uint4(hw[0], hw[1], hw[2], hw[3]);
  *reinterpret_cast<uint4*>(blk + 16 * (lane + 16)) = make_uint4(lw[0], lw[1], lw[2], lw[3]);
}

// ---- candidate lists in LDS ---------------------------------------------------
template <int NQ, int CAP>
struct Cand {
  uint64_t key[NQ][CAP];
  uint32_t idx[NQ][CAP];
  int cnt[NQ];
  uint64_t thr[NQ];
  int overflow;
};

// Selection over 64 PER entries held by one wave (empty slots: key 0, index
// 0xFFFFFFFF), of which at least topk are not empty: the entries to keep,
// exactly topk of them, are those with key > tk, or key == tk and idx <= ti. tk
// is found bit by bit from the top, the high word before the low one: the
// largest value that at least topk keys reach, stopping as soon as exactly topk
// do (then every key >= tk is kept). Only ballots of 32-bit comparisons and
// scalar counts, no barrier: about 25 rounds for scores.
template <int PER>
__device__ __forceinline__ void wave_select(const uint64_t (&key)[PER], const uint32_t (&idx)[PER],
                                            int topk, uint64_t& tk, uint32_t& ti) {
  uint32_t hi[PER];
#pragma unroll
  for (int j = 0; j < PER; ++j) hi[j] = (uint32_t)(key[j] >> 32);
  ti = 0xFFFFFFFFu;
  uint32_t t = 0;
  for (int b = 31; b >= 0; --b) {
    const uint32_t c = t | (1u << b);
    int n = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) n += __popcll(__ballot(hi[j] >= c));
    if (n >= topk) t = c;
    if (n == topk) {
      tk = (uint64_t)t << 32;
      return;
    }
  }
  // t is the high word of the topk-th key, and more than the missing entries share it
  int need = topk;
  uint32_t lo[PER];                          // low words of the entries with that high word
  bool in[PER];
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    need -= __popcll(__ballot(hi[j] > t));
    in[j] = hi[j] == t;
    lo[j] = (uint32_t)key[j];
  }
  uint32_t v = 0;
  for (int b = 31; b >= 0; --b) {
    const uint32_t c = v | (1u << b);
    int n = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) n += __popcll(__ballot(in[j] && lo[j] >= c));
    if (n >= need) v = c;
    if (n == need) {
      tk = ((uint64_t)t << 32) | v;
      return;
    }
  }
  tk = ((uint64_t)t << 32) | v;              // the topk-th key, shared: the smallest indices win
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    need -= __popcll(__ballot(in[j] && lo[j] > v));
    in[j] = in[j] && lo[j] == v;
  }
  uint32_t w = 0;                            // the need-th smallest index among them
  for (int b = 31; b >= 0; --b) {
    const uint32_t c = w | (1u << b);
    int n = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) n += __popcll(__ballot(in[j] && idx[j] < c));
    if (n < need) w = c;
  }
  ti = w;
}

// Writes the entries that wave_select keeps to key_o / idx_o (any order).
template <int PER>
__device__ __forceinline__ void wave_compact(const uint64_t (&key)[PER], const uint32_t (&idx)[PER],
                                             uint64_t tk, uint32_t ti, uint64_t* key_o,
                                             uint32_t* idx_o) {
  int base = 0;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const bool keep = key[j] > tk || (key[j] == tk && idx[j] <= ti);
    const uint64_t m = __ballot(keep);
    if (keep) {
      const int at = base + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
      key_o[at] = key[j];
      idx_o[at] = idx[j];
    }
    base += __popcll(m);
  }
}

// One wave prunes one list to its topk entries (in any order) and sets its
// threshold; a list of at most topk entries is left as it is. Entries past CAP
// (counted but not stored) are dropped here; their owners insert them again.
template <int CAP>
__device__ __forceinline__ void prune_list(uint64_t* key, uint32_t* idx, int* cnt, uint64_t* thr,
                                           int topk) {
  constexpr int PER = CAP / 64;
  const int lane = threadIdx.x & 63;
  const int c = __builtin_amdgcn_readfirstlane(min(*cnt, CAP));
  if (c < topk) {
    if (lane == 0) *cnt = c;
    return;
  }
  uint64_t k[PER];
  uint32_t id[PER];
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int e = 64 * j + lane;
    k[j] = e < c ? key[e] : 0ull;
    id[j] = e < c ? idx[e] : 0xFFFFFFFFu;
  }
  uint64_t tk;
  uint32_t ti;
  wave_select<PER>(k, id, topk, tk, ti);
  wave_lds_order();                          // every lane has read its entries
  wave_compact<PER>(k, id, tk, ti, key, idx);
  if (lane == 0) {
    *cnt = topk;
    *thr = tk;
  }
}
// Prunes every list of at least `least` entries, NWV lists at a time. Callers
// put a barrier before and after.
template <int NQ, int CAP, int NWV>
__device__ __forceinline__ void prune(Cand<NQ, CAP>& cd, int least, int topk) {
  for (int q = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)); q < NQ; q += NWV)
    if (__builtin_amdgcn_readfirstlane(cd.cnt[q]) >= least)
      prune_list<CAP>(cd.key[q], cd.idx[q], &cd.cnt[q], &cd.thr[q], topk);
}

struct ScoreArgs {
  const uint8_t* codes;
  int64_t cstride;
  const uint16_t* scales;
  int64_t N;
  int U;
  const ModInfo* mods;
  const uint4* planes;
  int n_steps;
  int64_t grp;
  const int32_t* fq;     // [groups][U][16]
  const int64_t* ysum;   // [groups][U][16]
  int64_t Q;
  int topk;
  float* full;
  uint64_t* ckey;   // [grid][NQ][topk], NQ = queries of the pass
  uint32_t* cidx;
  // multi-module pass: module ranges (range r = modules rng[r] .. rng[r+1]-1)
  // and the per-(module, query, row) integer dots it writes, [U][NQ][N]
  int n_rng;
  int32_t rng[MAX_RNG + 1];
  void* part;
  int64_t n_tiles;   // tiled store: 32-row tiles (ceil(N / 32))
};

// NQT: groups of 16 queries per pass. RT: 32-row tiles per wave. NCLS:
// accumulator classes of the bit expansion (1 or 2). MODE 0 / 3: one module (of
// at most / more than 2^16 bits: its dots fit 32 bits or take 64); its fp64 term
// is formed after the last step and the rows are offered to the per-query
// candidate lists. MODE 1 / 2: several modules; a work unit is
// (row block, range of modules), and at the end of each module the exact dot
// <y_int, 2b - 1> of every (row, query) is written to `part` as int32 (MODE 1,
// every k_u <= 2^16) or int64 (MODE 2); k_score_fold then forms the fp64 terms
// and sums them in module order. CAP: candidate slots per query (MODE 0).
// TILED: the store is in the tiled layout (see eogp_sign_pack_tiled): each
// wave's 32-row tile and step is one 2 KB block whose bytes are already in
// lane order, each half a contiguous 1 KB; else rows are row-major.
// WHOLE (row-major): the 64 bytes of a row that a step takes are requested together,
// a step ahead, not 32 bytes at a time.
template <int NQT, int RT, int NCLS, int MODE, int CAP, bool TILED, bool WHOLE = false>
__global__ __launch_bounds__(NTHR) __attribute__((amdgpu_waves_per_eu(2, 2)))
void k_score(ScoreArgs a) {
  constexpr bool MULTI = MODE == 1 || MODE == 2;
  typedef typename std::conditional<MODE == 3, int64_t, int32_t>::type dot_t;   // one module's dots
  constexpr int NQ = NQT * QB;
  constexpr int ROWS = NW * RT * 32;   // rows per block
  static_assert(NCLS == 1 || NCLS == 2, "bit-weight classes");
  static_assert(RT * NQT <= 8, "accumulator registers");
  // fragments read ahead of their use, so that at least 8 MFMAs cover the LDS latency
  constexpr int FD = RT * NQT >= 8 ? 1 : RT * NQT >= 4 ? 2 : 3;
  __shared__ __attribute__((aligned(16))) uint4 sP[2][NQT * HALF_U4];
  __shared__ Cand<MULTI ? 1 : NQ, MULTI ? 64 : CAP> cd;   // (unused by several modules)
  // the wave index through readfirstlane: wave-uniform for the compiler, so the
  // row and tile arithmetic that depends on it stays scalar
  const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r32 = lane & 31, hg = lane >> 5;
  const cptr<int32_t> cmods = (cptr<int32_t>)(a.mods);   // ModInfo fields, 4 per module
  const cptr<int32_t> cfq = (cptr<int32_t>)(a.fq);
  const cptr<int64_t> cys = (cptr<int64_t>)(a.ysum);
  if (!MULTI) {
    if (tid < NQ) {
      cd.cnt[tid] = 0;
      cd.thr[tid] = 0ull;
    }
    if (tid == 0) cd.overflow = 0;
    __syncthreads();
  }
  const int64_t n_blocks = (a.N + ROWS - 1) / ROWS;
  const uint32_t M1 = 0x01010101u;
  int shv[8];                          // the shift of round t
#pragma unroll
  for (int t = 0; t < 8; ++t) shv[t] = opaque_shift(t - t % NCLS);

  // Work units. MODE 0: row blocks at a fixed stride. Multi-module: units
  // (range, block) in range-major order, dealt to the XCDs in contiguous
  // chunks (workgroup b runs on XCD b % 8), so the workgroups of one XCD share
  // the plane fragments of few module ranges in their L2.
  const int nrng = MULTI ? a.n_rng : 1;
  const int64_t n_units = n_blocks * nrng;
  const int G = gridDim.x, b = blockIdx.x;
  const bool xq = MULTI && G >= kXcds && G % kXcds == 0;
  const int nq = xq ? kXcds : 1, xcd = xq ? b % kXcds : 0;
  const int64_t chunk = (n_units + nq - 1) / nq;
  const int64_t q_end = std::min<int64_t>((int64_t)(xcd + 1) * chunk, n_units);
  const int64_t u_first = (int64_t)xcd * chunk + b / nq, u_step = G / nq;

  // Where a walk over the steps of a unit stands (all uniform). n: steps of the
  // unit; s: step within it; the rest (several modules, or row-major rows): the
  // module, the step within it, its steps, bytes and first byte in a row.
  struct Walk {
    int64_t unit, blk;
    int n, s, s_lo, u, u_hi, sl, nst, kbytes, boff;
  };
  auto open_module = [&](Walk& w) __attribute__((always_inline)) {
    const int k = cmods[4 * w.u];
    w.sl = 0;
    w.nst = (k + 8 * SB - 1) / (8 * SB);
    w.kbytes = k >> 3;
    w.boff = cmods[4 * w.u + 2];
  };
  auto open_unit = [&](Walk& w, int64_t unit) __attribute__((always_inline)) {
    w.unit = unit;
    const int rg = MULTI ? (int)(unit / n_blocks) : 0;
    w.blk = MULTI ? unit % n_blocks : unit;
    w.u = MULTI ? a.rng[rg] : 0;
    w.u_hi = MULTI ? a.rng[rg + 1] : 1;
    w.s_lo = MULTI ? cmods[4 * w.u + 3] : 0;
    w.n = ((MULTI && w.u_hi < a.U) ? cmods[4 * w.u_hi + 3] : a.n_steps) - w.s_lo;
    w.s = 0;
    if (MULTI || !TILED) open_module(w);
  };
  auto next_step = [&](Walk& w) __attribute__((always_inline)) {   // within the unit
    ++w.s;
    if ((MULTI || !TILED) && ++w.sl == w.nst && ++w.u < w.u_hi) open_module(w);
  };

  if (u_first < q_end) {
    Walk wl, wc;   // the loads' walk and the products'
    // this wave's rows in the loads' block: tiled, the tile's first block of
    // the unit (uniform); row-major, this lane's row
    const uint8_t* lrow[RT];
    auto row_of = [&](int64_t blk, int rt) { return blk * ROWS + (int64_t)(wid * RT + rt) * 32 + r32; };
    auto load_unit = [&](int64_t unit) __attribute__((always_inline)) {
      open_unit(wl, unit);
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        if constexpr (TILED) {
          const int64_t tile = std::min<int64_t>(wl.blk * (ROWS / 32) + wid * RT + rt, a.n_tiles - 1);
          const uint64_t off = (uint64_t)((tile * a.n_steps + wl.s_lo) * 2048);
          lrow[rt] = a.codes + (((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(off >> 32)) << 32) |
                                (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)off));
        } else {
          lrow[rt] = a.codes + std::min<int64_t>(row_of(wl.blk, rt), a.N - 1) * a.cstride;
        }
      }
    };

    i32x16 acc[RT][NQT][NCLS];
    auto clear_acc = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int qt = 0; qt < NQT; ++qt)
#pragma unroll
          for (int w = 0; w < NCLS; ++w)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[rt][qt][w][r] = 0;
    };
    clear_acc();
    // Code words of the two halves of a step: each half requested again as soon as
    // it is used, or (WHOLE) both together into nx, a step ahead.
    uint4 cw[2][RT];
    uint4 nx[2][WHOLE ? RT : 1];
    // this thread's share of the next half's plane fragments (WHOLE: of each half's next)
    i32x4 pw[WHOLE ? 2 : 1][NQT];
    uint32_t s16[RT];     // one module: the rows' scales

    // Half H of the loads' step: the plane fragments (staged at the end of the next
    // half) before the code words (used after it), in the order they are
    // consumed, as the load counter completes in order.
    auto load_planes = [&](auto half_c) __attribute__((always_inline)) {
      constexpr int H = decltype(half_c)::value;
#pragma unroll
      for (int qt = 0; qt < NQT; ++qt)
        pw[WHOLE ? H : 0][qt] = reinterpret_cast<const i32x4*>(
            a.planes)[((((int64_t)a.grp + qt) * a.n_steps + wl.s_lo + wl.s) * FRAGS + 8 * H) * 64 + tid];
    };
    // Row-major rows whose module ends inside the half (k_u a multiple of 64
    // bits): each lane reads its 16 bytes as two pieces of 8, those outside the
    // module from readable bytes instead (the first piece, or the store's first
    // 8 bytes): the planes are zero there, so the loaded words are used as they are.
    auto load_codes = [&](auto half_c, uint4 (&to)[RT]) __attribute__((always_inline)) {
      constexpr int H = decltype(half_c)::value;
      if constexpr (TILED) {
        const int64_t so = (int64_t)wl.s * 2048 + H * 1024;
        const uint32_t lo = (uint32_t)lane * 16;
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) to[rt] = *reinterpret_cast<const uint4*>(lrow[rt] + so + lo);
      } else {
        const int at = SB * wl.sl + 32 * H + 16 * hg;           // within the module's bytes
        const int64_t pos = (int64_t)wl.boff + at;              // within the row
        if (SB * wl.sl + 32 * H + 32 <= wl.kbytes) {            // uniform
#pragma unroll
          for (int rt = 0; rt < RT; ++rt) to[rt] = *reinterpret_cast<const uint4*>(lrow[rt] + pos);
        } else {
          const int have = wl.kbytes - at;                      // multiple of 8
#pragma unroll
          for (int rt = 0; rt < RT; ++rt) {
            const uint8_t* p0 = have >= 8 ? lrow[rt] + pos : a.codes;
            const uint8_t* p1 = have >= 16 ? lrow[rt] + pos + 8 : p0;
            const uint2 v0 = *reinterpret_cast<const uint2*>(p0), v1 = *reinterpret_cast<const uint2*>(p1);
            to[rt] = make_uint4(v0.x, v0.y, v1.x, v1.y);
          }
          // keeps the two branches apart: merged, the 16-byte loads of whole
          // halves became one of 8 bytes and two of 4 each (473,050 rows of
          // 6,144 bits, 16 queries: 237 us merged, 186 us apart)
          asm volatile("" ::: "memory");
        }
      }
    };
    auto stage = [&](auto half_c) __attribute__((always_inline)) {
      constexpr int H = decltype(half_c)::value;
#pragma unroll
      for (int qt = 0; qt < NQT; ++qt)
        *reinterpret_cast<i32x4*>(&sP[H][qt * HALF_U4 + tid]) = pw[WHOLE ? H : 0][qt];
    };
    // the loads' walk moves on, into the next unit after the last step of this
    // one (past the last unit it stays, and its last step is read again, unused)
    auto advance_loads = [&]() __attribute__((always_inline)) {
      if (wl.s + 1 < wl.n) next_step(wl);
      else if (wl.unit + u_step < q_end) load_unit(wl.unit + u_step);
    };

    // n1 of (tile rt, group qt, query i of the lane's eight) from the classes
    auto class_sum = [&](int rt, int qt, int r) __attribute__((always_inline)) {
      int v = acc[rt][qt][0][r];
      if constexpr (NCLS == 2) v += acc[rt][qt][1][r] >> 1;
      return v;
    };
    // <y_int, 2b - 1> of (row, query): query 8 (i / 4) + 4 hg + i % 4 of group qt
    auto dot = [&](int rt, int qt, int i, int64_t ys) __attribute__((always_inline)) -> int64_t {
      const int64_t n1 = 256 * (int64_t)class_sum(rt, qt, i) + (int64_t)class_sum(rt, qt, i + 8);
      return 2 * n1 - ys;
    };
    // Several modules: the dots of module wc.u to `part`. A lane's eight sums of
    // y_int come as two scalar loads of 64 bytes and a select by arithmetic: a
    // select between two loads becomes one load per lane and sum, each waiting
    // for every request and store before it (30 modules of up to 1,536 bits,
    // 694,444 codes, one query: the pass 960 us, now 703). Pairs of queries past the
    // last are not written (76 modules of 256 bits, 285,916 codes, one query: the
    // call 1,004 us with them, 606 without).
    auto fold_module = [&]() __attribute__((always_inline)) {
      const int64_t upper = -(int64_t)hg;
#pragma unroll
      for (int qt = 0; qt < NQT; ++qt) {
        const int64_t mo = ((a.grp + qt) * a.U + wc.u) * QB;
        const int nq = (int)std::min<int64_t>(QB, a.Q - (a.grp + qt) * QB);   // queries of the group
        int64_t ys[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int64_t lo = cys[mo + 8 * (i >> 2) + (i & 3)], hi = cys[mo + 8 * (i >> 2) + (i & 3) + 4];
          ys[i] = lo ^ ((lo ^ hi) & upper);
        }
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
          const int64_t row = row_of(wc.blk, rt);
          auto put = [&](int i) __attribute__((always_inline)) {   // query q0 + 4 hg of the group
            const int q0 = 8 * (i >> 2) + (i & 3);
            const int64_t o = ((int64_t)wc.u * NQ + QB * qt + q0 + 4 * hg) * a.N + row;
            const int64_t nn = dot(rt, qt, i, ys[i]);
            if constexpr (MODE == 1) static_cast<int32_t*>(a.part)[o] = (int32_t)nn;
            else static_cast<int64_t*>(a.part)[o] = nn;
          };
          if (row < a.N) {
            if (nq == QB) {
#pragma unroll
              for (int i = 0; i < 8; ++i) put(i);
            } else {
#pragma unroll
              for (int i = 0; i < 8; ++i)
                if (8 * (i >> 2) + (i & 3) < nq) put(i);           // (uniform)
            }
          }
        }
      }
      clear_acc();
    };

    auto half_step = [&](auto half_c) __attribute__((always_inline)) {
      constexpr int H = decltype(half_c)::value;
      const uint4* frag = &sP[H][lane];
      i32x4 fr[FD + 1][NQT];
#pragma unroll
      for (int f = 0; f < FD; ++f)
#pragma unroll
        for (int qt = 0; qt < NQT; ++qt) fr[f][qt] = __builtin_bit_cast(i32x4, frag[qt * HALF_U4 + f * 64]);
      __builtin_amdgcn_sched_group_barrier(0x100, FD * NQT, 0);                // the first DS reads
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        if (t + FD < 8)
#pragma unroll
          for (int qt = 0; qt < NQT; ++qt)
            fr[(t + FD) % (FD + 1)][qt] = __builtin_bit_cast(i32x4, frag[qt * HALF_U4 + (t + FD) * 64]);
        const int w = t % NCLS, sh = t - w;
        const uint32_t mk = M1 << w;
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
          const uint4 c = cw[H][rt];
          // bits shifted across the halves land at 32 - sh and above, never
          // under the mask (its highest bit is 24 + w, and sh + w <= 7)
          uint64_t p0 = ((uint64_t)c.y << 32) | c.x, p1 = ((uint64_t)c.w << 32) | c.z;
          if (sh) {
            p0 >>= shv[t];
            p1 >>= shv[t];
          }
          i32x4 av;
          av[0] = (int)((uint32_t)p0 & mk);
          av[1] = (int)((uint32_t)(p0 >> 32) & mk);
          av[2] = (int)((uint32_t)p1 & mk);
          av[3] = (int)((uint32_t)(p1 >> 32) & mk);
#pragma unroll
          for (int qt = 0; qt < NQT; ++qt)
            acc[rt][qt][w] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fr[t % (FD + 1)][qt], av, acc[rt][qt][w], 0, 0, 0);
        }
        // per round: the fragment reads ahead, then each tile's expansion and MFMAs
        if (t + FD < 8) __builtin_amdgcn_sched_group_barrier(0x100, NQT, 0);   // DS read
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
          __builtin_amdgcn_sched_group_barrier(0x002, 6, 0);                   // VALU
          __builtin_amdgcn_sched_group_barrier(0x008, NQT, 0);                 // MFMA
        }
      }
    };
    constexpr std::integral_constant<int, 0> H0{};
    constexpr std::integral_constant<int, 1> H1{};

    auto load_half = [&](auto half_c) __attribute__((always_inline)) {
      load_planes(half_c);
      load_codes(half_c, cw[decltype(half_c)::value]);
    };
    // WHOLE: the next step's code words take their place, and the one after it is
    // requested. The copies are kept in front of the requests: made at the loop's
    // end instead, they wait for what was just requested.
    auto turn_over = [&]() __attribute__((always_inline)) {
      if constexpr (WHOLE) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int rt = 0; rt < RT; ++rt) {
            cw[h][rt] = nx[h][rt];
            asm volatile("" : "+v"(cw[h][rt].x), "+v"(cw[h][rt].y), "+v"(cw[h][rt].z), "+v"(cw[h][rt].w));
          }
        advance_loads();
        load_planes(H0);
        load_codes(H0, nx[0]);
        load_codes(H1, nx[1]);
      }
    };

    // prologue: step 0 requested (WHOLE: step 1's code words and first planes too),
    // its first half staged
    load_unit(u_first);
    load_half(H0);
    stage(H0);
    load_half(H1);
    advance_loads();
    if constexpr (WHOLE) {
      load_planes(H0);
      load_codes(H0, nx[0]);
      load_codes(H1, nx[1]);
    }
    __syncthreads();
    for (int64_t unit = u_first; unit < q_end; unit += u_step) {
      open_unit(wc, unit);
      if (!MULTI) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) s16[rt] = a.scales[std::min<int64_t>(row_of(wc.blk, rt), a.N - 1)];
      }
      for (int s = 0; s < wc.n; ++s) {
        half_step(H0);
        stage(H1);
        if constexpr (WHOLE) load_planes(H1);
        else load_half(H0);
        __syncthreads();
        half_step(H1);
        stage(H0);                     // the next step's (or the next unit's first) half
        if constexpr (WHOLE) turn_over();
        else load_half(H1);
        // (after the requests: the next waits would include its stores)
        if (MULTI && wc.sl == wc.nst - 1) fold_module();
        __syncthreads();
        next_step(wc);
        if constexpr (!WHOLE) advance_loads();
      }
      if constexpr (!MULTI) {
        // candidates of this block. The opaque copy of the lane half keeps the
        // list addresses from being computed once before the block loop and
        // held through it.
        int hq = hg;
        asm volatile("" : "+v"(hq));
        // the exact dots take the accumulators' place (half their registers)
        dot_t nd[RT][NQT][8];
#pragma unroll
        for (int qt = 0; qt < NQT; ++qt)
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const int64_t mo = (a.grp + qt) * QB + 8 * (i >> 2) + (i & 3);
            const int64_t ys = hq ? cys[mo + 4] : cys[mo];
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
              // (32-bit dots: the steps may wrap, the result fits)
              if constexpr (MODE == 3) nd[rt][qt][i] = dot(rt, qt, i, ys);
              else
                nd[rt][qt][i] = (int32_t)(2u * (256u * (uint32_t)class_sum(rt, qt, i) +
                                                (uint32_t)class_sum(rt, qt, i + 8)) - (uint32_t)ys);
            }
          }
        // f(qt, i, list, exponent) for the lane's queries. The dots pass through
        // an opaque step first: each walk forms its scores anew instead of
        // keeping them (two registers each) from one walk to the next.
        auto each_query = [&](auto&& f) __attribute__((always_inline)) {
#pragma unroll
          for (int qt = 0; qt < NQT; ++qt)
#pragma unroll
            for (int i = 0; i < 8; ++i) {
              const int i0 = 8 * (i >> 2) + (i & 3);
              const int64_t mo = (a.grp + qt) * QB + i0;
              const int fx = hq ? cfq[mo + 4] : cfq[mo];
#pragma unroll
              for (int rt = 0; rt < RT; ++rt) asm volatile("" : "+v"(nd[rt][qt][i]));
              f(qt, i, QB * qt + i0 + 4 * hq, fx);
            }
        };
        // s n, exact in fp64; the term is this times 2^-f
        auto product = [&](int rt, int qt, int i) __attribute__((always_inline)) {
          return (double)f16_bits_to_f32((uint16_t)s16[rt]) * (double)nd[rt][qt][i];
        };
        auto score = [&](int rt, int qt, int i, int f) __attribute__((always_inline)) {
          return ldexp(product(rt, qt, i), -f);
        };
        uint64_t pend = 0;
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
          if (row_of(wc.blk, rt) < a.N)
            for (int e = 0; e < 8 * NQT; ++e) pend |= 1ull << (8 * NQT * rt + e);
        if (unit == u_first) {
          // first block: the threshold from the lanes' maxima (256 rows' worth).
          // Lists past the last query keep theirs at zero: nothing is offered to
          // them, and their equal keys take every round of a selection (one
          // query over 256 codes of 128 bits: 38 us with them, 29 us without).
          each_query([&](int qt, int i, int qn, int fx) __attribute__((always_inline)) {
            uint64_t m = 0;
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
              const uint64_t key = order_key(score(rt, qt, i, fx));
              if ((pend >> (8 * NQT * rt)) & 1) m = key > m ? key : m;
            }
            cd.key[qn][wid * 32 + r32] = m;
          });
          __syncthreads();
          for (int q = wid; q < NQ && a.grp * QB + q < a.Q; q += NW) {
            uint64_t m[4];
            uint32_t id[4];
            int have = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              m[j] = cd.key[q][64 * j + lane];
              id[j] = 0;
              have += __popcll(__ballot(m[j] != 0));
            }
            if (have >= a.topk) {
              uint64_t tk;
              uint32_t ti;
              wave_select<4>(m, id, a.topk, tk, ti);
              if (lane == 0) cd.thr[q] = tk;
            }
          }
          __syncthreads();
        }
        if (a.full)
          each_query([&](int qt, int i, int qn, int fx) __attribute__((always_inline)) {
            const int64_t q = a.grp * QB + qn;
            if (q < a.Q)
#pragma unroll
              for (int rt = 0; rt < RT; ++rt) {
                const int64_t row = row_of(wc.blk, rt);
                if (row < a.N) a.full[q * a.N + row] = (float)score(rt, qt, i, fx);
              }
          });
        // a full list is pruned and the entries that did not fit are offered
        // again (the loop condition is uniform). Most products are below the
        // threshold times 2^f and need no more than that comparison; what is
        // not (NaN, or a threshold not set yet, included) is compared by key.
        for (;;) {
          each_query([&](int qt, int i, int qn, int fx) __attribute__((always_inline)) {
            const uint64_t thr = cd.thr[qn];
            const double least = ldexp(key_value(thr), fx);
            uint32_t may = 0;
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
              if (!(product(rt, qt, i) < least)) may |= 1u << rt;
            if (a.grp * QB + qn >= a.Q) may = 0;
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
              const uint64_t bit = 1ull << (8 * NQT * rt + 8 * qt + i);
              if ((may >> rt & 1) && (pend & bit)) {
                const uint64_t key = order_key(score(rt, qt, i, fx));
                if (key >= thr) {
                  const int pos = atomicAdd(&cd.cnt[qn], 1);
                  if (pos < CAP) {
                    cd.key[qn][pos] = key;
                    cd.idx[qn][pos] = (uint32_t)row_of(wc.blk, rt);
                    pend &= ~bit;
                  } else {
                    cd.overflow = 1;
                  }
                }
              }
            }
          });
          __syncthreads();
          const int ov = cd.overflow;
          __syncthreads();
          if (!ov) break;
          prune<NQ, CAP, NW>(cd, CAP, a.topk);
          if (tid == 0) cd.overflow = 0;
          __syncthreads();
        }
        clear_acc();
      }
    }
  }
  if constexpr (!MULTI) {
    // (the merge takes candidates in any order)
    __syncthreads();
    prune<NQ, CAP, NW>(cd, a.topk + 1, a.topk);
    __syncthreads();
    for (int i = tid; i < NQ * a.topk; i += NTHR) {
      const int qq = i / a.topk, e = i % a.topk;
      const int64_t o = ((int64_t)blockIdx.x * NQ + qq) * a.topk + e;
      const bool have = e < cd.cnt[qq];
      a.ckey[o] = have ? cd.key[qq][e] : 0ull;
      a.cidx[o] = have ? cd.idx[qq][e] : 0xFFFFFFFFu;
    }
  }
}

// Multi-module scores from the exact per-module dots: wave w of a workgroup
// takes queries 4w .. 4w+3 of the group for 64 consecutive stored rows (one
// per lane); for u = 0 .. U-1 in order, score += s_{i,u} * n * 2^-f (each
// term exact in fp64), then the rows are offered to the per-query candidate
// lists as in k_score. Workgroups walk blocks of 64 rows at a fixed stride;
// grid.y: the groups of 16 queries of the pass.
struct FoldArgs {
  const void* part;           // [U][NQ][N] int32 or int64
  const uint16_t* scales;     // [N][U] fp16 bits
  int64_t N;
  int U;
  const int32_t* fq;          // [groups][U][16]
  int64_t grp;                // first group of 16 queries of the pass; group grp + blockIdx.y here
  int nq;                     // NQ: queries of the pass
  int64_t Q;
  int topk;
  float* full;
  uint64_t* ckey;             // [grid.x][NQ][topk]
  uint32_t* cidx;
};
constexpr int FOLD_THR = 256;
constexpr int FOLD_QW = QB / (FOLD_THR / 64);   // queries per wave

template <int CAP, bool N64>
__global__ __launch_bounds__(FOLD_THR) void k_score_fold(FoldArgs a) {
  __shared__ Cand<QB, CAP> cd;
  const int tid = threadIdx.x, lane = tid & 63;
  const int q0 = __builtin_amdgcn_readfirstlane((tid >> 6) * FOLD_QW);   // wave-uniform
  const int64_t grp = a.grp + blockIdx.y;
  const cptr<int32_t> cfq = (cptr<int32_t>)(a.fq);
  // this wave's last query among its four (negative: it has none)
  const int last_q = (int)std::min<int64_t>(FOLD_QW, a.Q - (grp * QB + q0)) - 1;
  if (tid < QB) {
    cd.cnt[tid] = 0;
    cd.thr[tid] = 0ull;
  }
  if (tid == 0) cd.overflow = 0;
  __syncthreads();
  const int32_t* p32 = static_cast<const int32_t*>(a.part);
  const int64_t* p64 = static_cast<const int64_t*>(a.part);
  for (int64_t r0 = (int64_t)blockIdx.x * FOLD_ROWS; r0 < a.N;
       r0 += (int64_t)gridDim.x * FOLD_ROWS) {
    const int64_t row = r0 + lane;
    const bool ok = row < a.N;
    const int64_t rowc = ok ? row : a.N - 1;
    double sc[FOLD_QW];
#pragma unroll
    for (int j = 0; j < FOLD_QW; ++j) sc[j] = 0.0;
    // (queries past the last have no dots: their place in the wave reads those of its last)
#pragma unroll 4
    for (int u = 0; u < (last_q < 0 ? 0 : a.U); ++u) {
      const double sv = (double)f16_bits_to_f32(a.scales[rowc * a.U + u]);
      const int64_t mo = (grp * a.U + u) * QB + q0;
#pragma unroll
      for (int j = 0; j < FOLD_QW; ++j) {
        const int64_t o = ((int64_t)u * a.nq + blockIdx.y * QB + q0 + min(j, last_q)) * a.N + rowc;
        const int64_t nn = N64 ? p64[o] : (int64_t)p32[o];
        sc[j] += ldexp(sv * (double)nn, -cfq[mo + j]);
      }
    }
    uint32_t pend = 0;
#pragma unroll
    for (int j = 0; j < FOLD_QW; ++j) {
      const int64_t qg = grp * QB + q0 + j;
      if (ok && qg < a.Q) {
        if (a.full) a.full[qg * a.N + row] = (float)sc[j];
        pend |= 1u << j;
      }
    }
    for (;;) {
#pragma unroll
      for (int j = 0; j < FOLD_QW; ++j) {
        const uint32_t bit = 1u << j;
        const int q = q0 + j;
        if (pend & bit) {
          const uint64_t key = order_key(sc[j]);
          if (key < cd.thr[q]) {
            pend &= ~bit;
          } else {
            const int pos = atomicAdd(&cd.cnt[q], 1);
            if (pos < CAP) {
              cd.key[q][pos] = key;
              cd.idx[q][pos] = (uint32_t)row;
              pend &= ~bit;
            } else {
              cd.overflow = 1;
            }
          }
        }
      }
      __syncthreads();
      const int ov = cd.overflow;
      __syncthreads();
      if (!ov) break;
      prune<QB, CAP, FOLD_THR / 64>(cd, CAP, a.topk);
      if (tid == 0) cd.overflow = 0;
      __syncthreads();
    }
  }
  __syncthreads();
  prune<QB, CAP, FOLD_THR / 64>(cd, a.topk + 1, a.topk);
  __syncthreads();
  for (int i = tid; i < QB * a.topk; i += FOLD_THR) {
    const int qq = i / a.topk, e = i % a.topk;
    const int64_t o = ((int64_t)blockIdx.x * a.nq + blockIdx.y * QB + qq) * a.topk + e;
    const bool have = e < cd.cnt[qq];
    a.ckey[o] = have ? cd.key[qq][e] : 0ull;
    a.cidx[o] = have ? cd.idx[qq][e] : 0xFFFFFFFFu;
  }
}

// Reduction of the per-workgroup candidate lists ([G][NQ][topk] keys and
// indices, empty slots marked by index 0xFFFFFFFF) in two levels: workgroup
// (n, sp) merges lists sp * per .. sp * per + per - 1 of query n of the pass
// into one list of the same form (!FINAL, list sp of the output), then one
// workgroup per query merges those into the sorted top-k (FINAL). Each of the
// four waves selects the top-k of its share, up to 512 entries at a time in
// registers (wave_select), then the first wave selects among the four: no
// barrier but one between the two, and no more slots than topk per wave to look
// through (of 256 each, a merge of 24 lists of 10 took 13.1 + 8.6 us, now 10.1 +
// 7.4). Only the final top-k is put in order. (Before, a
// bitonic sort of up to 1,024 entries by the whole workgroup per 512 entries,
// one barrier per exchange stage: 49 + 46 us for the two levels at 256 lists of
// 100 for 16 queries, now 15 + 17 us for 32.)
constexpr int MRG_THR = 256, MRG_W = MRG_THR / 64, MRG_PER = 8;
struct MergeList {
  uint64_t key[MRG_W][MAX_TOPK];
  uint32_t idx[MRG_W][MAX_TOPK];
  int cnt[MRG_W];
};
// One wave: the top-k of the `total` entries that get(e, key, idx) yields
// (empty ones have index 0xFFFFFFFF) into key_o / idx_o; returns their number.
// key_o / idx_o may be read by get only at the same or a later entry than
// those already taken.
template <typename Get>
__device__ __forceinline__ int wave_topk(int total, int topk, uint64_t* key_o, uint32_t* idx_o,
                                         int kept, Get&& get) {
  const int lane = threadIdx.x & 63;
  for (int pos = 0; pos < total; pos += 64 * MRG_PER - kept) {
    // slots 0 .. kept - 1: the entries kept so far; then entries pos ..
    uint64_t key[MRG_PER];
    uint32_t id[MRG_PER];
    int have = 0;
#pragma unroll
    for (int j = 0; j < MRG_PER; ++j) {
      // every slot loads (a clamped entry where it has none), so that the
      // loads of all slots are in flight together
      const int slot = 64 * j + lane;
      const int e = pos + slot - kept;
      get(e < 0 ? 0 : e < total ? e : total - 1, key[j], id[j]);
      if (slot < kept) {
        key[j] = key_o[slot];
        id[j] = idx_o[slot];
      } else if (e >= total || id[j] == 0xFFFFFFFFu) {
        key[j] = 0ull;
        id[j] = 0xFFFFFFFFu;
      }
    }
#pragma unroll
    for (int j = 0; j < MRG_PER; ++j)
      have += __popcll(__ballot(id[j] != 0xFFFFFFFFu));
    const int before_kept = kept;
    uint64_t tk = 0;
    uint32_t ti = 0xFFFFFFFEu;               // every entry that is not empty
    if (have > topk) wave_select<MRG_PER>(key, id, topk, tk, ti);
    wave_lds_order();                        // every lane has read its slots
    wave_compact<MRG_PER>(key, id, tk, ti, key_o, idx_o);
    wave_lds_order();                        // the next round reads other lanes' entries
    kept = have < topk ? have : topk;
    pos += kept - before_kept;               // the loop adds 512 less the new count
  }
  return kept;
}
template <bool FINAL>
__global__ __launch_bounds__(MRG_THR, 1) void k_merge(const uint64_t* __restrict__ ckey,
                                                      const uint32_t* __restrict__ cidx, int G,
                                                      int per, int nq, int64_t grp, int64_t Q,
                                                      int topk, int64_t* __restrict__ out_idx,
                                                      float* __restrict__ out_score,
                                                      uint64_t* __restrict__ okey,
                                                      uint32_t* __restrict__ oidx) {
  __shared__ MergeList ml;
  const int n = blockIdx.x, sp = blockIdx.y;
  const int64_t q = grp * QB + n;
  if (q >= Q) return;                         // never read by the next level either
  const int tid = threadIdx.x, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l0 = sp * per, l1 = std::min(G, l0 + per);
  const int pw = (l1 - l0 + MRG_W - 1) / MRG_W;             // lists of this workgroup's waves
  const int w0 = std::min(l1, l0 + wid * pw), w1 = std::min(l1, w0 + pw);
  const int mine = wave_topk((w1 - w0) * topk, topk, ml.key[wid], ml.idx[wid], 0,
                             [&](int e, uint64_t& k, uint32_t& id) {
                               // (32-bit division: at most 512 lists of 256)
                               const uint32_t l = (uint32_t)e / (uint32_t)topk, at = (uint32_t)e - l * topk;
                               const int64_t o = ((int64_t)(w0 + l) * nq + n) * topk + at;
                               k = ckey[o];
                               id = cidx[o];
                             });
  if ((tid & 63) == 0) ml.cnt[wid] = mine;
  __syncthreads();
  if (wid == 0) {
    // the other waves' lists, as one row of MRG_W - 1 lists of topk slots
    const int c = wave_topk((MRG_W - 1) * topk, topk, ml.key[0], ml.idx[0], mine,
                            [&](int e, uint64_t& k, uint32_t& id) {
                              const int l = (int)((uint32_t)e / (uint32_t)topk), w = 1 + l, at = e - l * topk;
                              k = ml.key[w][at];
                              id = at < ml.cnt[w] ? ml.idx[w][at] : 0xFFFFFFFFu;
                            });
    if (tid == 0) ml.cnt[0] = c;
  }
  __syncthreads();
  const int c = ml.cnt[0];
  uint64_t* key = ml.key[0];
  uint32_t* idx = ml.idx[0];
  if constexpr (FINAL) {
    // each entry's place is the number of entries before it
    for (int e = tid; e < c; e += MRG_THR) {
      const uint64_t k = key[e];
      const uint32_t id = idx[e];
      int at = 0;
      for (int o = 0; o < c; ++o) at += before(key[o], idx[o], k, id) ? 1 : 0;
      out_idx[q * topk + at] = (int64_t)id;
      out_score[q * topk + at] = (float)key_value(k);
    }
    for (int e = c + tid; e < topk; e += MRG_THR) {
      out_idx[q * topk + e] = -1;
      out_score[q * topk + e] = -__builtin_inff();
    }
  } else {
    for (int e = tid; e < topk; e += MRG_THR) {
      const int64_t o = ((int64_t)sp * nq + n) * topk + e;
      okey[o] = e < c ? key[e] : 0ull;
      oidx[o] = e < c ? idx[e] : 0xFFFFFFFFu;
    }
  }
}

// One pass of nqt groups; MODE as in k_score.
template <int MODE, bool TILED>
void launch_pass(int nqt, int rt, dim3 gd, const ScoreArgs& a, hipStream_t s) {
  const dim3 bd(NTHR);
  if constexpr (MODE == 2 || MODE == 3) {
    hipLaunchKernelGGL((k_score<1, 2, 2, MODE, 512, TILED>), gd, bd, 0, s, a);
  } else {
    if constexpr (TILED) {   // (row-major stores take two tiles per wave)
      if (rt == 4) {
        if (nqt == 2) hipLaunchKernelGGL((k_score<2, 4, 1, MODE, 256, true>), gd, bd, 0, s, a);
        else hipLaunchKernelGGL((k_score<1, 4, 2, MODE, 512, true>), gd, bd, 0, s, a);
        return;
      }
    }
    // Row-major rows a multiple of 8 KB apart: lines of a row fall into few sets of the
    // L2 and are gone before the step's second half asks again (48 modules of 8,192 bits,
    // 20,000 codes: 1.6 times the fetches by halves), so whole steps are requested;
    // other rows by halves, which keeps more of the wait covered.
    if constexpr (MODE == 1 && !TILED) {
      if (a.cstride % 8192 == 0) {
        if (nqt == 2) hipLaunchKernelGGL((k_score<2, 2, 1, MODE, 256, false, true>), gd, bd, 0, s, a);
        else hipLaunchKernelGGL((k_score<1, 2, 2, MODE, 512, false, true>), gd, bd, 0, s, a);
        return;
      }
    }
    if (nqt == 2) hipLaunchKernelGGL((k_score<2, 2, 1, MODE, 256, TILED>), gd, bd, 0, s, a);
    else hipLaunchKernelGGL((k_score<1, 2, 2, MODE, 512, TILED>), gd, bd, 0, s, a);
  }
}

}  // namespace

int32_t score_max_topk() { return MAX_TOPK; }

// The least workspace a call runs with: the 16-query layout.
size_t score_ws_min(int64_t N, int64_t Q, int32_t U, const int64_t* kmod, int32_t topk) {
  return score_layout(N, Q, U, kmod, topk, PassCfg{1, 2}).total;
}
// The workspace of the pass that choose_cfg prefers.
size_t score_ws(int64_t N, int64_t Q, int32_t U, const int64_t* kmod, int32_t topk) {
  const PassCfg c = choose_cfg(N, Q, U, kmod, topk, true, ~size_t(0));
  return std::max(score_ws_min(N, Q, U, kmod, topk), score_layout(N, Q, U, kmod, topk, c).total);
}

template <bool TILED>
eogp_status score_topk_impl(const uint8_t* codes, int64_t cstride, const uint16_t* scales,
                            int64_t N, int32_t U, const int64_t* kmod, const float* Y, int64_t ldy,
                            int64_t Q, int32_t topk, int64_t* out_idx, float* out_score,
                            float* full, void* ws, size_t ws_bytes, hipStream_t s) {
  const PassCfg cfg = choose_cfg(N, Q, U, kmod, topk, TILED, ws_bytes);
  const ScoreLayout L = score_layout(N, Q, U, kmod, topk, cfg);
  if (ws_bytes < L.total) return fail(EOGP_ERR_WORKSPACE, "score_topk: workspace too small");
  if (Q == 0) return EOGP_OK;
  char* base = static_cast<char*>(ws);
  ModInfo* mods = reinterpret_cast<ModInfo*>(base + L.o_mods);
  int32_t* fq = reinterpret_cast<int32_t*>(base + L.o_fq);
  int64_t* ys = reinterpret_cast<int64_t*>(base + L.o_ys);
  int8_t* planes = reinterpret_cast<int8_t*>(base + L.o_pl);
  uint64_t* ck = reinterpret_cast<uint64_t*>(base + L.o_ck);
  uint32_t* ci = reinterpret_cast<uint32_t*>(base + L.o_ci);
  uint64_t* ck2 = reinterpret_cast<uint64_t*>(base + L.o_ck2);
  uint32_t* ci2 = reinterpret_cast<uint32_t*>(base + L.o_ci2);

  // the module table, MOD_CHUNK entries per launch (kernel arguments)
  int64_t coff = 0, boff = 0, sbase = 0;
  for (int u0 = 0; u0 < U; u0 += MOD_CHUNK) {
    ModChunk mc;
    mc.first = u0;
    mc.count = std::min(MOD_CHUNK, U - u0);
    for (int i = 0; i < mc.count; ++i) {
      const int64_t k = kmod[u0 + i];
      mc.m[i].k = (int32_t)k;
      mc.m[i].coff = (int32_t)coff;
      mc.m[i].boff = (int32_t)boff;
      mc.m[i].sbase = (int32_t)sbase;
      coff += k;
      boff += k / 8;
      sbase += (k + 8 * SB - 1) / (8 * SB);
    }
    hipLaunchKernelGGL(k_mod_table, dim3(1), dim3(MOD_CHUNK), 0, s, mc, mods);
  }
  EOGP_LAUNCH_CHECK("module table");
  timing::Scope tprep(EOGP_KT_SCORE_PREP, s);
  hipLaunchKernelGGL(k_query_stats, dim3((unsigned)(L.n_groups * QB), (unsigned)U), dim3(STAT_THR), 0,
                     s, Y, ldy, Q, U, mods, fq, ys);
  // one thread per 16 bytes of each of the two planes
  const int64_t pthreads = L.n_groups * L.n_steps * 512;
  hipLaunchKernelGGL(k_query_planes, dim3((unsigned)ceil_div(pthreads, 256)), dim3(256), 0, s, Y,
                     ldy, Q, U, mods, fq, L.n_steps, L.n_groups, TILED ? 1 : 0, planes);
  EOGP_LAUNCH_CHECK("query preparation");
  timing::end(tprep.slot, s);
  tprep.slot = -1;
  ScoreArgs a;
  a.codes = codes;
  a.cstride = cstride;
  a.scales = scales;
  a.N = N;
  a.U = U;
  a.mods = mods;
  a.planes = reinterpret_cast<const uint4*>(planes);
  a.n_steps = (int)L.n_steps;
  a.fq = fq;
  a.ysum = ys;
  a.Q = Q;
  a.topk = topk;
  a.full = full;
  a.ckey = ck;
  a.cidx = ci;
  a.n_rng = L.n_rng;
  a.part = base + L.o_part;
  a.n_tiles = ceil_div(N, 32);
  if (U > 1) module_ranges(kmod, U, L.n_steps, L.n_rng, a.rng);
  FoldArgs fa;
  fa.part = a.part;
  fa.scales = scales;
  fa.N = N;
  fa.U = U;
  fa.fq = fq;
  fa.Q = Q;
  fa.topk = topk;
  fa.full = full;
  fa.ckey = ck;
  fa.cidx = ci;
  for (int64_t grp = 0; grp < L.n_groups;) {
    const int nqt = cfg.nqt == 2 && grp + 1 < L.n_groups ? 2 : 1;   // an odd last group alone
    const int nq = nqt * QB;
    a.grp = grp;
    fa.grp = grp;
    fa.nq = nq;
    {
      // one pass over the store: the streaming kernel, and for several
      // modules the fold that adds their terms in order
      timing::Scope tp(EOGP_KT_SCORE_PASS, s);
      const dim3 gd((unsigned)L.grid);
      if (U == 1) {
        if (L.n64) launch_pass<3, TILED>(nqt, cfg.rt, gd, a, s);
        else launch_pass<0, TILED>(nqt, cfg.rt, gd, a, s);
      } else {
        if (L.n64) launch_pass<2, TILED>(nqt, cfg.rt, gd, a, s);
        else launch_pass<1, TILED>(nqt, cfg.rt, gd, a, s);
        const dim3 fg((unsigned)L.fold_grid, (unsigned)nqt), fb(FOLD_THR);
        if (fold_cap(topk) == 256) {
          if (L.n64) hipLaunchKernelGGL((k_score_fold<256, true>), fg, fb, 0, s, fa);
          else hipLaunchKernelGGL((k_score_fold<256, false>), fg, fb, 0, s, fa);
        } else {
          if (L.n64) hipLaunchKernelGGL((k_score_fold<512, true>), fg, fb, 0, s, fa);
          else hipLaunchKernelGGL((k_score_fold<512, false>), fg, fb, 0, s, fa);
        }
      }
    }
    timing::Scope tm(EOGP_KT_SCORE_MERGE, s);
    const int lists = (int)(U == 1 ? L.grid : L.fold_grid);
    const int sp = std::min(L.merge_split, std::max(1, lists / 8)), per = (int)ceil_div(lists, sp);
    if (sp > 1) {
      hipLaunchKernelGGL(k_merge<false>, dim3(nq, sp), dim3(MRG_THR), 0, s, ck, ci, lists, per, nq, grp,
                         Q, topk, nullptr, nullptr, ck2, ci2);
      hipLaunchKernelGGL(k_merge<true>, dim3(nq), dim3(MRG_THR), 0, s, ck2, ci2, sp, sp, nq, grp, Q,
                         topk, out_idx, out_score, nullptr, nullptr);
    } else {
      hipLaunchKernelGGL(k_merge<true>, dim3(nq), dim3(MRG_THR), 0, s, ck, ci, lists, lists, nq, grp, Q,
                         topk, out_idx, out_score, nullptr, nullptr);
    }
    EOGP_LAUNCH_CHECK("score pass");
    grp += nqt;
  }
  return EOGP_OK;
}

eogp_status score_topk(const uint8_t* codes, int64_t cstride, const uint16_t* scales, int64_t N,
                       int32_t U, const int64_t* kmod, const float* Y, int64_t ldy, int64_t Q,
                       int32_t topk, int64_t* out_idx, float* out_score, float* full, void* ws,
                       size_t ws_bytes, hipStream_t s) {
  return score_topk_impl<false>(codes, cstride, scales, N, U, kmod, Y, ldy, Q, topk, out_idx,
                                out_score, full, ws, ws_bytes, s);
}

eogp_status score_topk_tiled(const uint8_t* codes, const uint16_t* scales, int64_t N, int32_t U,
                             const int64_t* kmod, const float* Y, int64_t ldy, int64_t Q,
                             int32_t topk, int64_t* out_idx, float* out_score, float* full,
                             void* ws, size_t ws_bytes, hipStream_t s) {
  return score_topk_impl<true>(codes, 0, scales, N, U, kmod, Y, ldy, Q, topk, out_idx, out_score,
                               full, ws, ws_bytes, s);
}

// ---- scoring without a caller workspace ---------------------------------------
// For callers that cannot allocate device memory (code under graph capture,
// serving loops): the workspace of a scoring call lives in this file-scope
// array, one copy per GPU, held until the process ends. Its device address is
// looked up once per device, with that device current, and only that address
// is handed to kernels. Every call on one GPU shares the array, so calls that
// overlap on one GPU race; nothing in it has to start at zero (each call
// writes every byte it reads).
namespace {
constexpr size_t kScratchBytes = size_t(128) << 20;
static __device__ __align__(256) uint8_t scratch[kScratchBytes];
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

size_t score_scratch_bytes() { return kScratchBytes; }

eogp_status score_scratch(void** out) {
  int dev = 0;
  EOGP_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices)
    return fail(EOGP_ERR_UNSUPPORTED, "score_topk_noalloc: device index out of range");
  std::lock_guard<std::mutex> g(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return check_hip(e, "score_topk_noalloc: scratch address");
    if (!p) return fail(EOGP_ERR_DEVICE, "score_topk_noalloc: no scratch address");
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return EOGP_OK;
}

}  // namespace eogp
