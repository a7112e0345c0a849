// Device-side helpers shared by the gfx950 kernels: vector types, bf16 and
// OCP e4m3fn conversions, wavefront reductions, and the work-plan layout.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace rp {

// Tokens per KV page (the only page size the kernels are built for).
constexpr int kPage = 16;
// Pages per prefix work item, and the split of each response into work items:
// a response of P pages becomes floor(P / B) pieces of B pages and, if P is
// not a multiple of B, one ragged piece with the rest. Items are dispatched
// largest first (all B-sized pieces, then the ragged ones by decreasing
// size). The planner picks B per batch among kRespChunkStep, 2x, 3x and 4x
// that (32 to 128 pages): the multiple of kRespChunkStep nearest to
// W / (kRespChunkStep * kUnitsPerCu * compute units), W being the batch's
// response pages times its kv-heads, so that a batch has about kUnitsPerCu
// B-sized units per compute unit or more. Long pieces amortise each unit's
// start-up latency on big batches; small batches keep enough units in flight
// to fill the memory pipeline. Measured alternatives with extra small pieces
// at the end cost more start-ups than they saved. Batches whose work is below
// three quarters of one 32-page step take 16-page pieces instead, when the
// workspace was sized for them: a layout with at most
// kSmallBatchPageHeads page-heads of response capacity (sequences x table
// width x kv-heads) is sized for 16-page pieces, any other for 32.
constexpr int kPrefixChunkPages = 16;
constexpr int kRespChunkStep = 32;
constexpr int kRespChunkChoices = 4;
constexpr int kRespChunkPagesSmall = 16;
constexpr int kRespChunkPagesMin = kRespChunkStep;
constexpr int kRespChunkPagesMax = kRespChunkStep * kRespChunkChoices;
constexpr int kUnitsPerCu = 6;
constexpr long long kSmallBatchPageHeads = 1ll << 17;

constexpr float kLog2e = 1.4426950408889634f;
// Headroom of a lazily updated softmax running maximum, in log2 units: the
// maximum moves only when new scores exceed it by more than this, so the
// weights exp2(s - m) stay below 2^8 and most updates leave the output
// accumulator unscaled.
constexpr float kLazyMax = 8.0f;
constexpr float kLn2 = 0.6931471805599453f;

// Plan header slots.
enum : int {
  kHdrPrefixItems = 0,
  kHdrRespItems = 1,
  kHdrBigRespItems = 2,   // B-sized response items (they come first)
  kHdrRespChunkPages = 3,
  kHdrSlots = 16
};
// Largest group count the planner keeps in LDS.
constexpr int kPlanMaxGroups = 4096;
// Batches of at most this many sequences are planned by a single wave.
constexpr int kSmallPlanMaxSeqs = 64;
// Waves of a workgroup of the one-launch attention of small batches.
constexpr int kSmallWaves = 8;

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

__host__ __device__ inline int cdiv(int a, int b) { return (a + b - 1) / b; }

// Pointers into a planned workspace (all device memory). Partial results of
// query row r = s * Hq + j live in slots r * parts_per_row + k: first the
// group's prefix chunks (k < prefix chunks of the group), then the sequence's
// response chunks.
struct PlanView {
  int* hdr;            // [kHdrSlots]
  int* grp_off;        // [G+1] CSR of members
  int* grp_members;    // [S]   members of each group in ascending order of arrival
  int2* prefix_items;  // [max_prefix_items]  (group, chunk)
  int4* resp_items;    // [max_resp_items]    (sequence, first page, tokens, slot), longest first
  int* seq_parts;      // [S] partial results per query row of each sequence
  float* part_o;       // [S*Hq*parts_per_row][D]
  float* part_lse;     // [S*Hq*parts_per_row]
  int max_prefix_chunks;  // per group
  int max_resp_chunks;    // response items per sequence (at the smaller big-item length)
  int parts_per_row;      // max_prefix_chunks + max_resp_chunks
  int max_parts;          // capacity of part_o / part_lse
  int max_prefix_items;   // capacity of prefix_items
  int max_resp_items;     // capacity of resp_items
};

// Partial-result slot, kept inside the workspace even for a workspace that was
// never planned (garbage offsets then give garbage numbers, not stray writes).
__device__ inline int clamp_part(int p, int max_parts) {
  return (unsigned)p < (unsigned)max_parts ? p : 0;
}

// ---- bf16 ---------------------------------------------------------------
__device__ inline float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ inline float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// Two fp32 values to packed bf16 (low half first), round to nearest even, by
// gfx950's packed conversion (a NaN stays a NaN).
__device__ inline uint32_t pack_bf16x2(float lo, float hi) {
  typedef __bf16 bf16x2_v __attribute__((ext_vector_type(2)));
  typedef float f32x2_v __attribute__((ext_vector_type(2)));
  const f32x2_v v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_v));
}

// ---- OCP e4m3fn -----------------------------------------------------------
// Decoding is gfx950's conversion instructions, which implement OCP e4m3fn.

// fp32 -> e4m3fn code, round to nearest even, saturating at +-448. A NaN
// input (inf included among |x| >= 448) also takes the saturated code, with
// its sign bit: the append and page-write rules never store the NaN code.
__device__ inline uint32_t f32_to_e4m3(float x) {
  const uint32_t u = __float_as_uint(x);
  const uint32_t sign = (u >> 24) & 0x80u;
  const uint32_t a = u & 0x7FFFFFFFu;
  uint32_t code;
  if (a >= 0x43E00000u) {                 // |x| >= 448, inf or NaN
    code = 0x7Eu;
  } else if (a < 0x3C800000u) {           // |x| < 2^-6: subnormal grid of step 2^-9
    float q = __builtin_rintf(__uint_as_float(a) * 512.0f);  // exact scaling, RNE
    code = (uint32_t)q;                   // 0..8; 8 encodes 2^-6 exactly
  } else {
    const uint32_t e = (a >> 23) - 127u + 7u;   // 1..15 (2^-6 <= |x| < 448)
    const uint32_t m = a & 0x7FFFFFu;
    const uint32_t keep = m >> 20, rem = m & 0xFFFFFu;
    const uint32_t up = (rem > 0x80000u) || (rem == 0x80000u && (keep & 1u));
    code = (e << 3) + keep + up;          // a mantissa carry bumps the exponent
    if (code > 0x7Eu) code = 0x7Eu;
  }
  return code | sign;
}

// e4m3 codes of x[i] / scale, the quotient rounded to fp32 and then to e4m3 as
// f32_to_e4m3 does, four codes per word. inv = 1 / scale rounded; `plain`: no
// x[i] is NaN, |x[i]| <= 448 scale up to rounding, and scale is in
// plain_scale's range. A product with inv is then within 3 fp32 ulps of the
// quotient, so its e4m3 code is the quotient's unless it lies that close to
// the middle between two codes: 20 low mantissa bits near 0x80000, or near 0
// where the codes are subnormal. gfx950's conversion rounds to nearest even
// and equals f32_to_e4m3 on every fp32 value up to 464. Values that close, and
// those that are not plain, are divided.
// About 7 instructions a value against 26 (prefill of 32 x 1024 tokens into fp8
// pages: 239 us dividing every value, 222 this way).
__device__ inline bool plain_scale(float scale) { return scale >= 0x1p-100f && scale <= 0x1p100f; }
template <int N>
__device__ inline void e4m3_quotients(const float (&x)[N], float scale, float inv, bool plain, uint32_t (&w)[N / 4]) {
#pragma clang fp contract(off)
  static_assert(N % 4 == 0, "whole words");
  constexpr uint32_t kLow = 0xFFFFFu, kUlps = 4;
  uint32_t mid = 0xFFFFFFFFu;
  float q[N], least = INFINITY;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    q[i] = x[i] * inv;
    mid = min(mid, (__float_as_uint(q[i]) + 0x80000u + kUlps) & kLow);
    least = fminf(least, fabsf(q[i]));
  }
  bool divide = !plain || mid <= 2 * kUlps;
  if (least < 0x1p-6f) {
#pragma unroll
    for (int i = 0; i < N; ++i)
      divide = divide || (fabsf(q[i]) < 0x1p-6f && q[i] != 0.f && ((__float_as_uint(q[i]) + kUlps) & kLow) <= 2 * kUlps);
  }
#pragma unroll
  for (int k = 0; k < N / 4; ++k) {
    int v = __builtin_amdgcn_cvt_pk_fp8_f32(q[4 * k], q[4 * k + 1], 0, false);
    v = __builtin_amdgcn_cvt_pk_fp8_f32(q[4 * k + 2], q[4 * k + 3], v, true);
    w[k] = (uint32_t)v;
  }
  if (divide) {
#pragma unroll
    for (int k = 0; k < N / 4; ++k) {
      w[k] = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) w[k] |= f32_to_e4m3(x[4 * k + i] / scale) << (8 * i);
    }
  }
}

// ---- wavefront reductions -----------------------------------------------
template <int CTRL>
__device__ inline float dpp(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, false));
}
constexpr int kQuadSwap1 = 0xB1;     // quad_perm [1,0,3,2]
constexpr int kQuadSwap2 = 0x4E;     // quad_perm [2,3,0,1]
constexpr int kRowHalfMirror = 0x141;
constexpr int kRowMirror = 0x140;
constexpr int kRowShl = 0x100;       // + n: lane i of a row of 16 reads lane i + n

// Butterfly over the lanes that differ only in bits >= log2(FIRST) of the lane id.
template <int FIRST>
__device__ inline float xor_max_from(float x) {
#pragma unroll
  for (int o = FIRST; o < 64; o <<= 1) x = fmaxf(x, __shfl_xor(x, o));
  return x;
}
template <int FIRST>
__device__ inline float xor_sum_from(float x) {
#pragma unroll
  for (int o = FIRST; o < 64; o <<= 1) x += __shfl_xor(x, o);
  return x;
}

// Max over lanes l, l^16, l^32, l^48 (the four quads of an MFMA tile column)
// with gfx950's row-swap instructions, which stay in the VALU: swapping the
// halves (rows) of two copies of x puts x[l] and x[l^32] (x[l^16]) into the
// two results of every lane.
__device__ inline float max_xor16_32(float x) {
  const uint32_t u = __float_as_uint(x);
  const auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  x = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const uint32_t v = __float_as_uint(x);
  const auto b = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// Maxima over aligned groups of 16 lanes, over lanes l and l^16, and over the
// wave, in every lane, without the LDS crossbar.
__device__ inline float group_max16(float x) {
  x = fmaxf(x, dpp<kQuadSwap1>(x));
  x = fmaxf(x, dpp<kQuadSwap2>(x));
  x = fmaxf(x, dpp<kRowHalfMirror>(x));
  return fmaxf(x, dpp<kRowMirror>(x));
}
__device__ inline float max_xor16(float x) {
  const uint32_t v = __float_as_uint(x);
  const auto b = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ inline float wave_max(float x) { return max_xor16_32(group_max16(x)); }

// ---- the fp8 append rule --------------------------------------------------
// Row r of an fp8 (page, kv-head) block [16][D] takes a new token x. An
// aligned group of G lanes holds the row, N fp32 values (of bf16 inputs) a
// lane, in N / CH runs of CH consecutive columns: run k starts at col[k].
// `old` is the block's scale (its value does not matter for r = 0); `leader`
// marks the one lane that stores the new one. amax = max |x| over the row; row
// 0 sets scale = amax / 448 (1 when amax is 0); a later row keeps the old
// scale when amax <= 448 * old, and otherwise sets scale = amax / 448 and has
// rows 0..r-1 requantised from code * old: append_fp8_row returns that as a
// job, which requantise_fp8_rows must do next. Plain IEEE fp32 (no
// contraction, quotients as the division rounds them), so the bytes are a
// deterministic function of the inputs. Every lane of a G-lane group must call
// append_fp8_row, with the same r.
//
// The rule is a chain of memory round trips and then bound by the requantised
// values (about 12 instructions each), so callers load `old` early and the
// whole wave shares a block's rows, in 8-byte words: about one new row in
// seven raises its page's scale, so a wave mostly has one job or none, and the
// lanes of its other rows would wait. (Prep of 1024 sequences into fp8 pages:
// single bytes and a late scale 24.4 us, whole words by the row's own 16 lanes
// 13.3, this way 11.3.)
struct RequantJob {
  uint8_t* blk;
  float old, scale;
  int rows;  // 0: nothing to do
};

template <int CH, int N>
__device__ inline void put_codes(uint8_t* row, const int (&col)[N / CH], const uint32_t (&w)[N / 4]) {
#pragma unroll
  for (int k = 0; k < N / CH; ++k) {
    if constexpr (CH == 4) *reinterpret_cast<uint32_t*>(row + col[k]) = w[k];
    else *reinterpret_cast<uint16_t*>(row + col[k]) = (uint16_t)(w[k / 2] >> (16 * (k % 2)));
  }
}
template <int D, int G, int CH, int N>
__device__ RequantJob append_fp8_row(uint8_t* blk, float* scale_slot, float old, int r, const float (&x)[N],
                                     const int (&col)[N / CH], bool leader) {
#pragma clang fp contract(off)
  static_assert(G == 16 || G == 32, "lanes per row");
  static_assert(CH == 4 || (CH == 2 && N % 4 == 0), "columns per run");
  float amax = 0.f;
  bool plain = true;  // no NaN element
#pragma unroll
  for (int e = 0; e < N; ++e) {
    amax = fmaxf(amax, fabsf(x[e]));
    plain = plain && x[e] == x[e];
  }
  amax = group_max16(amax);
  if constexpr (G == 32) amax = max_xor16(amax);
  RequantJob job = {blk, old, old, 0};
  if (r == 0) {
    job.scale = amax > 0.f ? amax / 448.0f : 1.0f;
  } else if (!(amax <= 448.0f * old)) {
    job.scale = amax / 448.0f;
    job.rows = r;
  }
  uint32_t w[N / 4];
  e4m3_quotients(x, job.scale, 1.0f / job.scale, plain && plain_scale(job.scale), w);
  put_codes<CH, N>(blk + (size_t)r * D, col, w);
  if (leader) *scale_slot = job.scale;
  return job;
}

// Does the jobs of the lanes marked `leader`, one after the other, with every
// lane of the wave (all of them must call it): the next job's rows are loaded
// while one is requantised.
template <int D>
__device__ inline void requantise_fp8_rows(const RequantJob& job, bool leader, int lane) {
#pragma clang fp contract(off)
  constexpr int LPR = D / 8, RPI = 64 / LPR, LOADS = kPage / RPI;  // lanes per row, rows per load, loads per block
  unsigned long long todo = __ballot(leader && job.rows > 0);
  if (todo == 0) return;
  const int row0 = lane / LPR, off = lane * 8;
  const auto blk_of = [&](int src) __attribute__((always_inline)) {
    const uint64_t p = reinterpret_cast<uint64_t>(job.blk);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)p, src);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(p >> 32), src);
    return reinterpret_cast<uint8_t*>((uint64_t)hi << 32 | lo) + off;
  };
  const auto load = [&](int src, uint2 (&c)[LOADS]) __attribute__((always_inline)) {
    const uint8_t* b = blk_of(src);
    const int rows = __builtin_amdgcn_readlane(job.rows, src);
#pragma unroll
    for (int i = 0; i < LOADS; ++i)
      if (row0 + i * RPI < rows) c[i] = *reinterpret_cast<const uint2*>(b + i * RPI * D);
  };
  uint2 cur[LOADS] = {}, next[LOADS] = {};
  int src = __builtin_ctzll(todo);
  load(src, cur);
  while (true) {
    todo &= todo - 1;
    const int after = todo != 0 ? __builtin_ctzll(todo) : -1;
    if (after >= 0) load(after, next);
    uint8_t* b = blk_of(src);
    const int rows = __builtin_amdgcn_readlane(job.rows, src);
    const float old = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(job.old), src));
    const float scale = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(job.scale), src));
    const float inv = 1.0f / scale;
    const bool scales = plain_scale(scale) && plain_scale(old);
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
      if (row0 + i * RPI >= rows) continue;
      const uint32_t c[2] = {cur[i].x, cur[i].y};
      float y[8];
      uint32_t nan = 0;  // bytes with the NaN code carry into their top bit
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        nan |= (c[k] & 0x7F7F7F7Fu) + 0x01010101u;
        const auto lo = __builtin_amdgcn_cvt_pk_f32_fp8((int)c[k], false);
        const auto hi = __builtin_amdgcn_cvt_pk_f32_fp8((int)c[k], true);
        y[4 * k] = lo[0] * old;
        y[4 * k + 1] = lo[1] * old;
        y[4 * k + 2] = hi[0] * old;
        y[4 * k + 3] = hi[1] * old;
      }
      uint32_t w[2];
      e4m3_quotients(y, scale, inv, scales && (nan & 0x80808080u) == 0, w);
      *reinterpret_cast<uint2*>(b + i * RPI * D) = make_uint2(w[0], w[1]);
    }
    if (after < 0) return;
    src = after;
#pragma unroll
    for (int i = 0; i < LOADS; ++i) cur[i] = next[i];
  }
}

// MFMA tiles of the decode and prefill attention (fp32 accumulate).
// With lane l = 16 q + r (r < 16):
//   16x16x32 bf16: lane (r, q) supplies A[r][8q..8q+7] and B[8q..8q+7][r];
//   16x16x16 bf16: lane (r, q) supplies A[r][4q..4q+3] and B[4q..4q+3][r];
// lane (r, q) receives C[4q..4q+3][r].
// rp_selftest_mfma checks each of these against a matrix product.
__device__ inline f32x4_t mfma16x16x32(const bf16x8_t& a, const bf16x8_t& b, const f32x4_t& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
__device__ inline f32x4_t mfma16x16x16(const bf16x4_t& a, const bf16x4_t& b, const f32x4_t& c) {
  typedef short s16x4_t __attribute__((ext_vector_type(4)));
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4_t, a), __builtin_bit_cast(s16x4_t, b),
                                                   c, 0, 0, 0);
}

// gfx950's transposing LDS read (ds_read_b64_tr_b16): within each 16-lane
// group, lane s supplies the address of 4 consecutive 16-bit elements, and
// lane j receives element j % 4 of the elements addressed by lanes j / 4,
// 4 + j / 4, 8 + j / 4 and 12 + j / 4, in that order. With lane s pointing at
// row r0 + s / 4, columns c0 + 4 (s % 4) ... + 3 of a row-major tile, lane j
// receives rows r0 .. r0 + 3 of column c0 + j.
__device__ inline bf16x4_t lds_read_tr(const uint16_t* p) {
  typedef short s16x4_t __attribute__((ext_vector_type(4)));
  return __builtin_bit_cast(
      bf16x4_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t*)(p)));
}

__device__ inline float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ inline float fast_log2(float x) { return __builtin_amdgcn_logf(x); }

}  // namespace rp
