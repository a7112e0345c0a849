// Shared-prefix prefill. Every response of a GRPO group is sampled from the
// same prompt, so the prompt is processed once per group: its K/V are written
// into the group's prefix pages (the pages every response then reads while
// decoding) and its tokens attend causally within the prompt.
//
// K/V write: one wave per (group, prefix page, kv-head). bf16 pools copy the
// rows; fp8 pools get, in plain IEEE fp32, scale = amax / 448 over the page's
// written rows (1 when amax = 0) and codes e4m3(x / scale), round to nearest
// even, saturating.
//
// Causal attention: a workgroup of 4 waves per (group, kv-head, block of
// query rows); a 16-row tile holds 16 / n_rep consecutive prompt tokens times
// the n_rep query heads that share the kv-head, so every key block serves all
// of them (details at the kernel). K/V are read from the projections (not
// from the pool), as the prompt's own attention needs no quantised copy.
#include "rp_device.h"
#include "rp_internal.h"

namespace rp {
namespace {

// Length and first packed row of group g's prompt, clamped to the table width
// and to the packed arrays.
__device__ inline int prompt_len(const PrefillArgs& a, int g, int* first) {
  const int o0 = min(max(a.prompt_offs[g], 0), a.num_tokens);
  const int o1 = min(max(a.prompt_offs[g + 1], o0), a.num_tokens);
  *first = o0;
  return min(o1 - o0, a.max_prefix_pages * kPage);
}

// ---------------------------------------------------------------------------
// K/V page write
// ---------------------------------------------------------------------------
// One (page, kv-head) block of an fp8 pool from `rows` token rows by one wave:
// the rows stay in registers between the maximum and the codes. Magnitudes of
// bf16 values compare as integers; a NaN (above infinity) takes the maximum
// over the others in fp32.
template <int D>
struct Fp8Head {
  static constexpr int CPR = D / 8;            // 8-element chunks per row
  static constexpr int NC = kPage * CPR / 64;  // chunks per lane
  uint32_t v[NC][4];

  __device__ inline void load(const uint16_t* src, size_t src_row_pitch, int rows, int lane) {
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      const int c = lane + i * 64, r = c / CPR, col = (c % CPR) * 8;
      uint4 w = make_uint4(0, 0, 0, 0);
      if (r < rows) w = *reinterpret_cast<const uint4*>(src + (size_t)r * src_row_pitch + col);
      v[i][0] = w.x;
      v[i][1] = w.y;
      v[i][2] = w.z;
      v[i][3] = w.w;
    }
  }

  __device__ inline void store(uint8_t* blk, float* scale_slot, int rows, int lane) const {
#pragma clang fp contract(off)
    typedef uint16_t u16x2_t __attribute__((ext_vector_type(2)));
    u16x2_t top = {0, 0};
#pragma unroll
    for (int i = 0; i < NC; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        top = __builtin_elementwise_max(top, __builtin_bit_cast(u16x2_t, v[i][e] & 0x7FFF7FFFu));
    const uint32_t m = top[0] > top[1] ? top[0] : top[1];
    float amax = __uint_as_float(m << 16);
    const bool nan = __any(m > 0x7F80u);
    if (nan) {
      amax = 0.f;
#pragma unroll
      for (int i = 0; i < NC; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) amax = fmaxf(amax, fmaxf(fabsf(bf16_lo(v[i][e])), fabsf(bf16_hi(v[i][e]))));
    }
    amax = wave_max(amax);
    const float scale = amax > 0.f ? amax / 448.0f : 1.0f;
    const float inv = 1.0f / scale;
    const bool plain = !nan && plain_scale(scale);
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      const int c = lane + i * 64, r = c / CPR, col = (c % CPR) * 8;
      float x[8];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        x[2 * e] = bf16_lo(v[i][e]);
        x[2 * e + 1] = bf16_hi(v[i][e]);
      }
      uint32_t codes[2];
      e4m3_quotients(x, scale, inv, plain, codes);
      if (r < rows) *reinterpret_cast<uint2*>(blk + (size_t)r * D + col) = make_uint2(codes[0], codes[1]);
    }
    if (lane == 0) *scale_slot = scale;
  }
};

template <int D, bool FP8>
__global__ __launch_bounds__(64) void prefill_kv_write_kernel(const PrefillArgs a) {
  const int Hkv = a.num_kv_heads;
  const int b = blockIdx.x;
  const int h = b % Hkv;
  const int p = (b / Hkv) % a.max_prefix_pages;
  const int g = b / (Hkv * a.max_prefix_pages);
  int first;
  const int P = prompt_len(a, g, &first);
  const int rows = min(kPage, P - p * kPage);
  if (rows <= 0) return;
  const int page = clamp_page(a.prefix_block_table[(size_t)g * a.max_prefix_pages + p], a.num_pages);
  const int lane = threadIdx.x;
  const size_t pitch = (size_t)Hkv * D;  // elements between consecutive tokens of the projections
  const size_t src0 = (size_t)(first + p * kPage) * pitch + (size_t)h * D;
  const uint16_t* ks = static_cast<const uint16_t*>(a.k) + src0;
  const uint16_t* vs = static_cast<const uint16_t*>(a.v) + src0;
  const size_t blk = ((size_t)page * Hkv + h) * kPage * D;  // in elements
  if constexpr (!FP8) {
    constexpr int CPR = D / 8;
    uint16_t* kd = static_cast<uint16_t*>(a.k_pages) + blk;
    uint16_t* vd = static_cast<uint16_t*>(a.v_pages) + blk;
    for (int c = lane; c < rows * CPR; c += 64) {
      const int r = c / CPR, col = (c - r * CPR) * 8;
      *reinterpret_cast<uint4*>(kd + (size_t)r * D + col) = *reinterpret_cast<const uint4*>(ks + r * pitch + col);
      *reinterpret_cast<uint4*>(vd + (size_t)r * D + col) = *reinterpret_cast<const uint4*>(vs + r * pitch + col);
    }
  } else {
    const size_t sidx = (size_t)page * Hkv + h;
    Fp8Head<D> kh, vh;
    kh.load(ks, pitch, rows, lane);
    vh.load(vs, pitch, rows, lane);
    kh.store(static_cast<uint8_t*>(a.k_pages) + blk, a.k_scale + sidx, rows, lane);
    vh.store(static_cast<uint8_t*>(a.v_pages) + blk, a.v_scale + sidx, rows, lane);
  }
}

// ---------------------------------------------------------------------------
// Causal attention
// ---------------------------------------------------------------------------
// Workgroup of 4 waves on (group, kv-head) pair and a block of query rows:
// wave w holds RT 16-row tiles (each 16 / n_rep consecutive prompt tokens
// times the n_rep query heads of the kv-head), so a workgroup covers
// 64 RT / n_rep tokens. Keys go through LDS in blocks of 32, copied there
// straight from the projections, with one barrier per block: two blocks ahead
// in three stages with two row tiles (three workgroups per compute unit, by
// registers and by LDS), one ahead in two stages with one (four). Per block
// and row tile: S^T = K Q^T on mfma 16x16x32 (Q stays in registers), a causal
// mask, one online-softmax update per row, and O^T += V^T P^T, also on mfma
// 16x16x32 (all 32 keys per instruction).
//
// What bounds it: with short prompts HBM and the start of each workgroup (32
// prompts of U[64, 512] tokens: 50 us, 3.0 TB/s with the pages), with long
// ones the softmax beside the matrix products (8 prompts of 2048-4096 tokens:
// 320 us, 1.0 PFLOP/s). Against staging through registers, the direct copies
// measured 8% (1024 tokens: 4%), the maximum inside the product 4%, the mask
// without a test for rows past the end 2%, and the order of pf_unit 12-20%.
enum PfPages { kPagesNone = 0, kPagesBf16 = 1, kPagesFp8 = 2 };  // what the attention kernel writes besides
constexpr int kPfWaves = 4;
constexpr int kPfThreads = 64 * kPfWaves;
constexpr int kKeyBlk = 32;

// A staged block holds K and V rows as they come from the projections, copied
// by direct global-to-LDS loads: one instruction of one wave fills a 1 KiB
// chunk of kRows rows. Row r lies in chunk r % kChunks, slot r / kChunks, and
// chunks are 32 bytes more than 1 KiB apart, so that the eight rows of a
// 16-byte K read and the four rows of a transposing V read lie in different
// banks (no conflict cycles by the counters), at offsets that are immediates of
// the reads.
template <int D>
struct PfSmem {
  static constexpr int kRows = 512 / D;                 // rows per chunk
  static constexpr int kChunks = kKeyBlk / kRows;       // chunks of a K (or V) block
  static constexpr int kPitch = 512 + 16;               // bf16 elements between chunks
  static constexpr int kElems = kChunks * kPitch;       // a K (or V) block
  static constexpr int kStage = 2 * kElems;
  static constexpr int kPerWave = 2 * kChunks / kPfWaves;  // copies per wave and block
  static_assert(kChunks % kPfWaves == 0, "chunks per wave");
  __device__ static constexpr int row(int r) { return (r % kChunks) * kPitch + (r / kChunks) * D; }
};
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

// One direct global-to-LDS copy by a whole wave: 16 bytes per lane from
// base + off to lds + 16 * lane. Written in assembly because the compiler
// waits for every load in flight before any LDS read that follows its own
// form of it; pf_wait waits for as many as are needed.
__device__ inline void pf_copy(uint32_t lds, const uint16_t* base, uint32_t off) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               :
               : "s"(lds), "v"(off), "s"(base)
               : "m0", "memory");
}
// Waits until at most N of the wave's copies are in flight (and its LDS reads
// are done), then for the workgroup's other waves.
template <int N>
__device__ inline void pf_wait() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"(N) : "memory");
}

// This wave's copies of one key block. Byte offsets within one prompt's rows
// fit 32 bits (the host checks it). Rows at or past the prompt's end are read
// from its last token (inside the packed arrays); their scores are masked.
template <int D>
__device__ inline void pf_load(uint32_t stage, const uint16_t* kbase, const uint16_t* vbase, uint32_t pitch, int u0,
                               int last, int wave, int lane) {
  using L = PfSmem<D>;
  const int slot = lane / (D / 8), col = (lane % (D / 8)) * 8;
#pragma unroll
  for (int i = 0; i < L::kPerWave / 2; ++i) {
    const int chunk = wave * (L::kPerWave / 2) + i;
    const uint32_t off = ((uint32_t)min(u0 + slot * L::kChunks + chunk, last) * pitch + (uint32_t)col) * 2u;
    pf_copy(stage + (uint32_t)(chunk * L::kPitch * 2), kbase, off);
    pf_copy(stage + (uint32_t)((L::kElems + chunk * L::kPitch) * 2), vbase, off);
  }
}

// Which (group, kv-head) pair and row block a workgroup takes. Workgroups are
// dealt to the 8 XCDs round-robin, so with NP a multiple of 8 all row blocks
// of a pair run on one XCD, and the order keeps few pairs at a time there: sets
// of `per_set`, their row blocks interleaved, the last rows (which see the most
// keys) first. Their keys then stay in the XCD's L2 (all pairs at once instead
// of five: 1024-token prompts 239 us against 198, 2048-4096 tokens 366 against
// 320). An XCD deals its workgroups to its shader engines in turn as well: an
// odd number of slots in a set (one idle where its pairs are even) and an odd
// `stride` from set to set keep a pair, or a row block, from falling to one
// engine every time (4 pairs instead of 5 on ragged prompts of 300-1800 tokens:
// 317 us against 208; last sets of 4 pairs, 9 prompts of 59-1127 tokens at Hq
// 64, Hkv 8: 120 us without the idle slot, 90 with).
// stride = 0: any NP, pairs dealt in turn, which is also the order of small
// grids.
constexpr int kPfPairs = 5;
// Pairs per set: all of an XCD's at once where they are few and their K and V
// fit the L2s together; the last set, which starts its longest rows when the
// others run dry, is otherwise a large part of such a grid (Hkv 8, d 128, us,
// sets of 5 against one: 9 prompts of 59-1127 tokens at Hq 32 59.5, 49.5; 6 of
// 100-1500 64.1, 51.0; 8 of 512-1024 62.6, 53.4. 32 or 64 pairs: 32 of U[64,
// 256] 30.8, 33.8; 64 of U[32, 128] 28.2, 29.3).
constexpr int kPfFewPairs = 16;
__host__ inline int pf_set_pairs(long long pairs, long long kv_bytes) {
  return pairs <= kPfFewPairs && kv_bytes <= (24ll << 20) ? (int)pairs : kPfPairs;
}
// Grids up to this many workgroups start nearly all of them at once (four 128-
// wide or six 64-wide workgroups with one row tile fit a compute unit): there
// is little left to keep in L2, and the long row blocks of all pairs first
// spread best over the compute units. Measured, pairs in turn against a few at
// a time, in us (Hq / Hkv, d, prompts; workgroups):
//   8 / 8, 128, 32 x U[32, 128]; 512:    10.3, 11.4;  16 x U[300, 400]; 896: 19.8, 21.2
//   16 / 8, 128, 32 x U[32, 128]; 1024:  13.2, 12.7;  16 x U[300, 400]; 1664: 27.3, 28.2
//   16 / 8, 128, 64 x U[64, 256]; 4096:  41.6, 36.3;  64 / 8, 8 x U[512, 1024]; 4096: 112, 101
//   16 / 8, 64, 32 x U[16, 64]; 512:     5.88, 6.29;  64 x U[32, 128]; 2048: 11.4, 12.0
// and against one set of few pairs:
//   32 / 8, 128, 4 x 600; 608:           24.4, 25.9;  64, 4 x U[1000, 2000]; 2016: 63.5, 52.3
//   8 / 8, 128, 12 x U[59, 1127]; 864:   34.5, 37.2;  16 / 8, 64, 8 x U[100, 1500]; 1536: 40.4, 35.2
__host__ inline long long pf_small_grid(long long pairs, int head_dim) {
  return pairs <= kPfFewPairs ? 1024 : 1024 * 128 / head_dim;
}
__device__ inline bool pf_unit(int b, int NP, int max_blocks, int stride, int per_set, int* pair, int* rb) {
  if (stride == 0) {
    *pair = b % NP;
    *rb = max_blocks - 1 - b / NP;
    return true;
  }
  const int i = b / 8, set = i / stride, r = i - set * stride;
  const int m = min(per_set, NP / 8 - set * per_set), odd = m | 1;  // pairs of this set
  *rb = max_blocks - 1 - r / odd;
  *pair = (set * per_set + r % odd) * 8 + b % 8;
  return *rb >= 0 && r % odd < m;
}

// The one-launch prefill writes a prompt's K/V rows into the group's prefix
// pages once a workgroup's attention is done: no register or wait of the key
// loop is spent on them. bf16 rows are written by the workgroup whose query
// rows hold the token (exactly one), fp8 pages, whose scale needs all their
// rows, by the one that holds the page's first token. Rows past the prompt's
// end are not written, as in the page-write kernel. (fp8, 32 prompts of
// U[64, 512]: a page-write launch before the attention 69 us in all, together
// 55.)
//
// bf16 rows come from LDS with one row tile per wave, where the last two key
// blocks hold them all, and from L2 with two (32 prompts of U[128, 256] at Hq 8,
// Hkv 8 from L2 19.2 us, from LDS 17.9; at 32 kv-heads 81.8, 74.3). Short
// prompts run every instruction once, so what is fetched counts: the loops are
// not unrolled and end with the prompt (4 prompts of U[16, 64] at Hq 8, Hkv 8:
// unrolled 6.25 us, rolled 5.80).
template <int D, int TPB>
__device__ inline void pf_write_pages_fp8(const PrefillArgs& a, int g, int h, int T0, int last, int wave, int lane,
                                          const uint16_t* kbase, const uint16_t* vbase, uint32_t pitch) {
  const int p0 = cdiv(T0, kPage), p1 = cdiv(min(T0 + TPB, last + 1), kPage);
  // A wave takes whole pages, K and V, where there is one for every wave, and
  // K or V of a page otherwise.
  constexpr int SPLIT = TPB / kPage >= kPfWaves ? 1 : 2;
  for (int task = wave; task < SPLIT * (p1 - p0); task += kPfWaves) {
    const int p = p0 + task / SPLIT, rows = min(kPage, last + 1 - p * kPage);
    const int page = clamp_page(a.prefix_block_table[(size_t)g * a.max_prefix_pages + p], a.num_pages);
    const size_t slot = (size_t)page * a.num_kv_heads + h, src = (size_t)p * kPage * pitch, dst = slot * (kPage * D);
    Fp8Head<D> head[3 - SPLIT];
    const bool v_only = SPLIT == 2 && (task & 1);
    head[0].load((v_only ? vbase : kbase) + src, pitch, rows, lane);
    if constexpr (SPLIT == 1) head[1].load(vbase + src, pitch, rows, lane);
    head[0].store(static_cast<uint8_t*>(v_only ? a.v_pages : a.k_pages) + dst, (v_only ? a.v_scale : a.k_scale) + slot,
                  rows, lane);
    if constexpr (SPLIT == 1) head[1].store(static_cast<uint8_t*>(a.v_pages) + dst, a.v_scale + slot, rows, lane);
  }
}

// From LDS: `last_blk` is the stage of key block `blk`, the workgroup's last,
// `prev_blk` that of the block before.
template <int D, int TPB>
__device__ inline void pf_write_staged(const PrefillArgs& a, int g, int h, int T0, int last, int t, int blk,
                                       const uint16_t* last_blk, const uint16_t* prev_blk) {
  using L = PfSmem<D>;
  static_assert(TPB <= 2 * kKeyBlk, "the workgroup's rows are staged");
  const int* pbt = a.prefix_block_table + (size_t)g * a.max_prefix_pages;
  const int n = min(TPB, last + 1 - T0) * (D / 8);
#pragma unroll 1
  for (int c = t; c < n; c += kPfThreads) {
    const int col = (c % (D / 8)) * 8, u = T0 + c / (D / 8);
    const uint16_t* src = (u / kKeyBlk == blk ? last_blk : prev_blk) + L::row(u % kKeyBlk) + col;
    const int page = clamp_page(pbt[u / kPage], a.num_pages);
    const size_t dst = (((size_t)page * a.num_kv_heads + h) * kPage + (u % kPage)) * D + col;
    *reinterpret_cast<u32x4_t*>(static_cast<uint16_t*>(a.k_pages) + dst) = *reinterpret_cast<const u32x4_t*>(src);
    *reinterpret_cast<u32x4_t*>(static_cast<uint16_t*>(a.v_pages) + dst) =
        *reinterpret_cast<const u32x4_t*>(src + L::kElems);
  }
}

template <int D, int TPB>
__device__ inline void pf_write_pages(const PrefillArgs& a, int g, int h, int T0, int last, int t,
                                      const uint16_t* kbase, const uint16_t* vbase, uint32_t pitch) {
  const int* pbt = a.prefix_block_table + (size_t)g * a.max_prefix_pages;
  const int n = min(TPB, last + 1 - T0) * (D / 8);  // 16-byte pieces of the workgroup's rows (K or V)
#pragma unroll 1
  for (int c = t; c < n; c += kPfThreads) {
    const int col = (c % (D / 8)) * 8, u = T0 + c / (D / 8);
    const size_t src = (size_t)u * pitch + col;
    const u32x4_t k = *reinterpret_cast<const u32x4_t*>(kbase + src), v = *reinterpret_cast<const u32x4_t*>(vbase + src);
    const int page = clamp_page(pbt[u / kPage], a.num_pages);
    const size_t dst = (((size_t)page * a.num_kv_heads + h) * kPage + (u % kPage)) * D + col;
    *reinterpret_cast<u32x4_t*>(static_cast<uint16_t*>(a.k_pages) + dst) = k;
    *reinterpret_cast<u32x4_t*>(static_cast<uint16_t*>(a.v_pages) + dst) = v;
  }
}

// One 32-key block from LDS stage `kst` (keys u0 .. u0 + 31) for this wave's
// RT row tiles: the scores of both 16-key sub-tiles, the causal mask, one
// online-softmax update per row for the whole block, then O^T += V^T P^T.
// The products start from minus the row's running maximum (mneg, in raw
// scores), so a block needs no cross-lane step unless some score exceeds that
// maximum by more than thr (kLazyMax in log2 units; minus infinity until the
// row has a maximum): then the maximum moves and the accumulator is rescaled.
// MASK = false for blocks that lie wholly at or below the diagonal of every
// row of the wave.
template <int D, int NREP, int RT, bool MASK>
__device__ __forceinline__ void pf_compute(const uint16_t* kst, int u0, float qk_scale, float thr_set, int r16,
                                           int quad, const int (&tr)[RT], const bf16x8_t (&qop)[RT][D / 32],
                                           f32x4_t (&oacc)[RT][D / 16], f32x4_t (&mneg)[RT], float (&thr)[RT],
                                           float (&lrow)[RT]) {
  using L = PfSmem<D>;
  constexpr int KB = D / 32, DT = D / 16, ST = kKeyBlk / 16;
  const uint16_t* vst = kst + L::kElems;
  // Entry i of sub-tile st: key u0 + st*16 + quad*4 + i against row r16.
  f32x4_t sacc[RT][ST];
  bf16x8_t kop[ST][KB];
#pragma unroll
  for (int st = 0; st < ST; ++st)
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
      kop[st][kb] = __builtin_bit_cast(
          bf16x8_t, *reinterpret_cast<const uint4*>(kst + L::row(r16) + L::row(st * 16) + kb * 32 + quad * 8));
  // The waves of a SIMD come from different workgroups and drift in and out
  // of phase; raising the priority of a wave while it issues its MFMAs lets
  // another wave's softmax fill the matrix core's shadow instead of
  // competing for issue slots (config-2 prompts 58.3 -> 54.2 us; prompts
  // of 512-2048 tokens, with two row tiles per wave, unchanged).
  __builtin_amdgcn_s_setprio(1);
#pragma unroll
  for (int st = 0; st < ST; ++st) {
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) sacc[rt][st] = mneg[rt];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) sacc[rt][st] = mfma16x16x32(kop[st][kb], qop[rt][kb], sacc[rt][st]);
  }
  __builtin_amdgcn_s_setprio(0);
  const uint16_t* vtr = vst + L::row(quad * 4 + r16 / 4) + 4 * (r16 % 4);
  const auto read_vop = [&](int dt) __attribute__((always_inline)) {
    const bf16x4_t v0 = lds_read_tr(vtr + dt * 16);
    const bf16x4_t v1 = lds_read_tr(vtr + L::row(16) + dt * 16);
    return __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7);
  };
  // With one row tile per wave there are registers to request the V^T
  // operands ahead of the softmax; with two they are read inside P V, one
  // 16-column tile at a time, which keeps three waves per SIMD.
  bf16x8_t vpre[DT];
  if constexpr (RT == 1) {
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) vpre[dt] = read_vop(dt);
    __builtin_amdgcn_sched_barrier(0);
  }
  bf16x4_t pop[RT][ST];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    float mx = -INFINITY;
#pragma unroll
    for (int st = 0; st < ST; ++st)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        // Rows past the prompt's end need no mask: they are not stored.
        if constexpr (MASK) sacc[rt][st][i] = st * 16 + i <= tr[rt] - u0 - quad * 4 ? sacc[rt][st][i] : -INFINITY;
        mx = fmaxf(mx, sacc[rt][st][i]);
      }
    if (__any(mx > thr[rt])) {
      mx = max_xor16_32(mx);
      const float up = mx > thr[rt] ? mx : 0.f;
      // A row's first maximum may be far below zero: nothing to rescale yet.
      const float alpha = thr[rt] == -INFINITY ? 0.f : fast_exp2(-up * qk_scale);
      thr[rt] = mx > thr[rt] ? thr_set : thr[rt];
      mneg[rt] -= up;
      lrow[rt] *= alpha;
#pragma unroll
      for (int st = 0; st < ST; ++st) sacc[rt][st] -= up;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) oacc[rt][dt] *= alpha;
    }
    float psum = 0.f;
#pragma unroll
    for (int st = 0; st < ST; ++st) {
      float pw[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) pw[i] = fast_exp2(sacc[rt][st][i] * qk_scale);
      psum += (pw[0] + pw[1]) + (pw[2] + pw[3]);
      pop[rt][st] =
          __builtin_bit_cast(bf16x4_t, make_uint2(pack_bf16x2(pw[0], pw[1]), pack_bf16x2(pw[2], pw[3])));
    }
    lrow[rt] += psum;
  }
  // O^T += V^T P^T over all 32 keys in one mfma 16x16x32 per 16 output
  // columns: lane (r16, quad) supplies contraction slots 8 quad .. 8 quad + 7,
  // taken as keys quad*4 .. quad*4 + 3 and 16 + quad*4 .. 16 + quad*4 + 3 in
  // both operands (any key order serves, as long as V^T and P^T share it).
  // The V^T operand of lane (r16, quad) is column dt*16 + r16 of those keys:
  // two transposing reads, in which lane s of the quad's 16 points at row
  // quad*4 + s/4 (then 16 rows further on), columns dt*16 + 4 (s % 4) ...+3.
  static_assert(ST == 2, "two 16-key sub-tiles per block");
  bf16x8_t pop8[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
    pop8[rt] = __builtin_shufflevector(pop[rt][0], pop[rt][1], 0, 1, 2, 3, 4, 5, 6, 7);
  __builtin_amdgcn_s_setprio(1);
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) {
    const bf16x8_t vo = RT == 1 ? vpre[dt] : read_vop(dt);
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) oacc[rt][dt] = mfma16x16x32(vo, pop8[rt], oacc[rt][dt]);
  }
  __builtin_amdgcn_s_setprio(0);
}

// Register budget: one row tile per wave fits four waves per SIMD (128
// VGPRs), two row tiles three (168 VGPRs).
template <int D, int NREP, int RT, PfPages WP>
__global__ __launch_bounds__(kPfThreads) __attribute__((amdgpu_waves_per_eu(RT == 1 ? 4 : 3, 8)))
void prefill_attn_kernel(const PrefillArgs a, int max_blocks, int stride, int per_set) {
  using L = PfSmem<D>;
  constexpr int KB = D / 32;              // MFMA k-blocks over head_dim
  constexpr int DT = D / 16;              // 16-column output tiles
  constexpr int TPT = 16 / NREP;          // prompt tokens per 16-row tile
  constexpr int TPW = RT * TPT;           // prompt tokens per wave
  constexpr int TPB = kPfWaves * TPW;     // prompt tokens per workgroup
  constexpr int STAGES = RT == 2 ? 3 : 2;
  __shared__ __attribute__((aligned(16))) uint16_t smem[STAGES * L::kStage];

  const int Hkv = a.num_kv_heads, Hq = a.num_q_heads;
  const int NP = a.num_groups * Hkv;
  int pair, rb;
  if (!pf_unit((int)blockIdx.x, NP, max_blocks, stride, per_set, &pair, &rb)) return;
  const int g = pair / Hkv, h = pair - g * Hkv;
  int first;
  const int P = prompt_len(a, g, &first);
  const int T0 = rb * TPB;
  if (T0 >= P) return;  // uniform over the workgroup
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6, r16 = lane & 15, quad = lane >> 4;
  const int last = P - 1;
  const size_t qpitch = (size_t)Hq * D, kpitch = (size_t)Hkv * D;
  const uint16_t* kbase = static_cast<const uint16_t*>(a.k) + (size_t)first * kpitch + (size_t)h * D;
  const uint16_t* vbase = static_cast<const uint16_t*>(a.v) + (size_t)first * kpitch + (size_t)h * D;

  // Row r16 of row tile rt: token T0 + wave * TPW + rt * TPT + r16 / NREP,
  // query head h * NREP + r16 % NREP. Q is the B operand of S^T = K Q^T.
  const int jr = h * NREP + r16 % NREP;
  int tr[RT];
  bf16x8_t qop[RT][KB];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    tr[rt] = T0 + wave * TPW + rt * TPT + r16 / NREP;
    const uint16_t* qrow = static_cast<const uint16_t*>(a.q) + (size_t)(first + min(tr[rt], last)) * qpitch +
                           (size_t)jr * D + quad * 8;
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
      qop[rt][kb] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4*>(qrow + kb * 32));
  }

  const int tlast = min(T0 + TPB, P) - 1;  // the workgroup's last token bounds its keys
  const int w_first = T0 + wave * TPW;  // this wave's first token
  const int nblk = tlast / kKeyBlk + 1;
  const float thr_set = kLazyMax / a.qk_scale;
  float thr[RT], lrow[RT];
  f32x4_t mneg[RT];
  f32x4_t oacc[RT][DT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    thr[rt] = -INFINITY;
    mneg[rt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    lrow[rt] = 0.f;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) oacc[rt][dt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  }

  // At a block's start its copies are complete (the wave's own, then, past
  // the barrier, everyone's); with three stages the next block's are in
  // flight, and the one after that is requested into the stage the barrier
  // has freed. With two stages the next block is requested then, except the
  // second, which goes into the stage that is free from the start (32 prompts
  // of U[16, 64] at Hq 16, Hkv 8, d 64: 5.6 us without, 5.4 with).
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint16_t*)smem;
  const int uwave = __builtin_amdgcn_readfirstlane(wave);
  const auto request = [&](int blk, int stage) __attribute__((always_inline)) {
    pf_load<D>(lds0 + (uint32_t)(stage * L::kStage * 2), kbase, vbase, (uint32_t)kpitch, blk * kKeyBlk, last, uwave,
               lane);
  };
  request(0, 0);
  // The compiler's wait for the q rows belongs here: it does not count the
  // copies, so inside the loop it would drain them in every block.
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) asm volatile("" : "+v"(qop[rt][kb]));
  if (nblk > 1) request(1, 1);
  int cur = 0;
  for (int blk = 0; blk < nblk; ++blk) {
    if ((STAGES == 3 || blk == 0) && blk + 1 < nblk) pf_wait<L::kPerWave>();
    else pf_wait<0>();
    if ((STAGES == 3 || blk > 0) && blk + STAGES - 1 < nblk) request(blk + STAGES - 1, cur == 0 ? STAGES - 1 : cur - 1);
    const uint16_t* kst = smem + cur * L::kStage;
    // Blocks wholly below the diagonal for every row of the wave skip the mask.
    if ((blk + 1) * kKeyBlk - 1 <= w_first)
      pf_compute<D, NREP, RT, false>(kst, blk * kKeyBlk, a.qk_scale, thr_set, r16, quad, tr, qop, oacc, mneg, thr,
                                     lrow);
    else
      pf_compute<D, NREP, RT, true>(kst, blk * kKeyBlk, a.qk_scale, thr_set, r16, quad, tr, qop, oacc, mneg, thr,
                                    lrow);
    cur = cur == STAGES - 1 ? 0 : cur + 1;
  }

  if constexpr (WP == kPagesBf16 && RT == 1)  // `cur` is past the last block's stage
    pf_write_staged<D, TPB>(a, g, h, T0, last, t, nblk - 1, smem + (1 - cur) * L::kStage, smem + cur * L::kStage);
  else if constexpr (WP == kPagesBf16)
    pf_write_pages<D, TPB>(a, g, h, T0, last, t, kbase, vbase, (uint32_t)kpitch);

#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const float lt = xor_sum_from<16>(lrow[rt]);
    if (tr[rt] > last) continue;
    const float inv = 1.f / lt;
    uint16_t* orow = static_cast<uint16_t*>(a.out) + (size_t)(first + tr[rt]) * qpitch + (size_t)jr * D + quad * 4;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      const f32x4_t v = oacc[rt][dt] * inv;
      *reinterpret_cast<uint2*>(orow + dt * 16) = make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
    }
    if (a.lse != nullptr && quad == 0)
      a.lse[(size_t)(first + tr[rt]) * Hq + jr] = (fast_log2(lt) - mneg[rt][0] * a.qk_scale) * kLn2;
  }
  if constexpr (WP == kPagesFp8)
    pf_write_pages_fp8<D, TPB>(a, g, h, T0, last, uwave, lane, kbase, vbase, (uint32_t)kpitch);
}

// Row tiles per wave: two when prompts average 384 tokens or more (each K/V
// operand read from LDS serves two MFMAs), one otherwise (twice the
// workgroups, which balances ragged short prompts better). Measured, one tile
// against two, in us at Hkv 8 (Hq, d, prompts):
//   16, 128, 32 x U[192, 320]: 32.1, 36.0;  32 x U[300, 400]: 45.1, 49.4
//   16, 128, 64 x 400: 121.5, 114.7;        32 x U[700, 900]: 168.9, 147.6
//   64, 128, 32 x U[300, 400]: 164.8, 148.7;  32, 64, 64 x 400: 121.2, 103.5
//   16, 128, 2 x 500: 12.5, 17.9;           1 x 1000: 19.8, 27.6
// A grid that fills the chip more than once gains by two tiles from about 300
// (many query heads) to 500 tokens (few) on, a smaller one at no length.
template <int D, int NREP>
hipError_t attn_launch(const PrefillArgs& a, hipStream_t st) {
  const long long NP = (long long)a.num_groups * a.num_kv_heads;
  const int max_tokens = a.max_prefix_pages * kPage;
  const int rt = (long long)a.num_tokens >= 384ll * a.num_groups ? 2 : 1;
  const int tpb = kPfWaves * rt * (16 / NREP);
  const int max_blocks = cdiv(max_tokens, tpb);
  // A launch has at most 2^24 workgroups of 256 threads; the idle ones of the
  // ordered grid must not be what exceeds it.
  int stride = 0, per_set = 0;
  long long blocks = NP * max_blocks;
  const long long pairs = NP / 8;  // of an XCD
  if (NP % 8 == 0 && blocks > pf_small_grid(pairs, D)) {
    const int n = pf_set_pairs(pairs, (long long)a.num_tokens * a.num_kv_heads * D * 4);
    const long long step = ((long long)(n | 1) * max_blocks) | 1, rest = pairs % n;
    const long long with_idle = 8 * (pairs / n * step + (rest == 0 ? 0 : rest | 1) * max_blocks);
    if (with_idle < (1ll << 24)) {
      per_set = n;
      stride = (int)step;
      blocks = with_idle;
    }
  }
  if (blocks <= 0) return hipSuccess;
  const dim3 grid((unsigned)blocks), block(kPfThreads);
  if (a.write_pages && a.k_scale != nullptr) {
    if (rt == 2) prefill_attn_kernel<D, NREP, 2, kPagesFp8><<<grid, block, 0, st>>>(a, max_blocks, stride, per_set);
    else prefill_attn_kernel<D, NREP, 1, kPagesFp8><<<grid, block, 0, st>>>(a, max_blocks, stride, per_set);
  } else if (a.write_pages) {
    if (rt == 2) prefill_attn_kernel<D, NREP, 2, kPagesBf16><<<grid, block, 0, st>>>(a, max_blocks, stride, per_set);
    else prefill_attn_kernel<D, NREP, 1, kPagesBf16><<<grid, block, 0, st>>>(a, max_blocks, stride, per_set);
  } else {
    if (rt == 2) prefill_attn_kernel<D, NREP, 2, kPagesNone><<<grid, block, 0, st>>>(a, max_blocks, stride, per_set);
    else prefill_attn_kernel<D, NREP, 1, kPagesNone><<<grid, block, 0, st>>>(a, max_blocks, stride, per_set);
  }
  return hipGetLastError();
}

template <int D>
hipError_t attn_by_nrep(const PrefillArgs& a, int n_rep, hipStream_t st) {
  switch (n_rep) {
    case 1: return attn_launch<D, 1>(a, st);
    case 2: return attn_launch<D, 2>(a, st);
    case 4: return attn_launch<D, 4>(a, st);
    case 8: return attn_launch<D, 8>(a, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_prefill_kv_write(const PrefillArgs& a, int head_dim, bool fp8, hipStream_t stream) {
  const long long blocks = (long long)a.num_groups * a.max_prefix_pages * a.num_kv_heads;
  if (blocks <= 0) return hipSuccess;
  const dim3 grid((unsigned)blocks), block(64);
  if (head_dim == 128) {
    if (fp8) prefill_kv_write_kernel<128, true><<<grid, block, 0, stream>>>(a);
    else prefill_kv_write_kernel<128, false><<<grid, block, 0, stream>>>(a);
  } else if (head_dim == 64) {
    if (fp8) prefill_kv_write_kernel<64, true><<<grid, block, 0, stream>>>(a);
    else prefill_kv_write_kernel<64, false><<<grid, block, 0, stream>>>(a);
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_prefill_attn(const PrefillArgs& a, int head_dim, int n_rep, hipStream_t stream) {
  if (head_dim == 128) return attn_by_nrep<128>(a, n_rep, stream);
  if (head_dim == 64) return attn_by_nrep<64>(a, n_rep, stream);
  return hipErrorInvalidValue;
}

}  // namespace rp
