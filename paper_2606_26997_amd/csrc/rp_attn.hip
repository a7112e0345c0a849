// Partial attention over planned work items, in one launch. Work units are
// (item, kv-head) pairs, one per one-wave block: all group-prefix units first,
// then the response units longest first, so the hardware dispatcher hands the
// last free slots the smallest units.
//
// Group-prefix units: every response of a GRPO group is sampled from the same
// prompt, so the group's prompt-prefix KV is read once per (group, kv-head,
// chunk) and applied to all of the group's query rows at once: live members x
// (Hq / Hkv) query heads, 16 rows per pass.
// Response units: one (sequence, chunk of response pages, kv-head), Hq / Hkv
// query rows.
//
// Both walk their pages on the matrix cores (attend_pages):
//   S^T  = K Q^T   on mfma 16x16x32 bf16 (M = 16 tokens, N = 16 columns, K = 32 of head_dim)
//   O^T += V^T P^T on mfma 16x16x16 or 16x16x32 bf16 (M = 16 head_dim columns, N = 16 columns)
// with fp32 accumulation and an online softmax. A response has at most 8
// query rows for the 16 columns, so its rows are repeated, and the copies of
// a row carry the three bf16 terms of its fp32 probabilities, whose sum keeps
// all 24 bits. How responses split into items is the planner's choice for the
// batch.
//
// Both are bound by HBM: a read of random 4 KiB blocks of a K and a V pool in
// equal units, with nothing computed, reaches 6.8 TB/s on an MI355X. Units of
// the sizes below reach 6.2 (256 sequences of up to 4096 tokens, where the
// launch's end counts most) to 6.65 TB/s (512 of up to 16384), whatever the
// occupancy (6 to 16 waves per compute unit) and the pages in flight per wave
// (one to three steps). With scores and P V on the VALU, as dot products and
// multiply-adds per query row, the response path was bound by its instructions
// from four query rows per kv-head on: 256 sequences of up to 8192 tokens at
// Hq 32, Hkv 4: 549 us a step against 398; at Hq 32, Hkv 8, d 64: 224 against
// 200; at Hq 16, Hkv 8 the two are equal.
//
// Each unit writes one partial (o normalised, lse natural-log) per query row
// into its fixed slot (row, chunk); the combine kernel merges a row's parts.
#include <type_traits>

#include "rp_device.h"
#include "rp_internal.h"
#include "rp_plan_small.h"

namespace rp {
namespace {

// V pages of responses are read with the non-temporal hint and K pages without
// it: both streams are read exactly once, and marking one of the two (either one) as
// streaming was measured 6-8% faster on every workload than marking neither
// or both.
// Loaded pages are held in clang vectors: HIP's uint4 is copied through
// memory-like moves that made each load wait for the one before it.
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
__device__ inline u32x4_t load_v_stream(const char* p) {
  return __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(p));
}

// Orders this wave's LDS accesses (its staging area is its own).
__device__ inline void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// 8 e4m3 codes -> 8 bf16 values (exact: every e4m3 value is a bf16 value), by
// gfx950's scaled conversion with scale 1: two codes per instruction.
template <bool HIGH>
__device__ inline uint32_t e4m3x2_to_bf16x2(uint32_t w) {
  return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, 1.0f, HIGH));
}
__device__ inline u32x4_t e4m3x8_to_bf16x8(uint32_t w0, uint32_t w1) {
  return u32x4_t{e4m3x2_to_bf16x2<false>(w0), e4m3x2_to_bf16x2<true>(w0), e4m3x2_to_bf16x2<false>(w1),
                 e4m3x2_to_bf16x2<true>(w1)};
}

// Geometry of one step of a unit: kPages pages whose K and V blocks are 4 KiB
// each in all, so every head size and element type has 8 KiB in flight per
// wave.
template <int D, bool FP8>
struct Geom {
  static constexpr int EB = FP8 ? 1 : 2;                 // bytes per KV element
  static constexpr int ROW_BYTES = D * EB;
  static constexpr int BLOCK_BYTES = kPage * ROW_BYTES;  // one (page, kv-head) block
  static constexpr int EPL = 16 / EB;                    // elements per 16-byte piece
  static constexpr int LOADS = BLOCK_BYTES / 1024;       // pieces per lane and block
  static constexpr int PAGES = 4 / LOADS;                // pages per step
  static constexpr int TOKENS = PAGES * kPage;
  static constexpr int PITCH = D + 16;                   // staged V row (bf16): the rows of a transposing read meet no bank twice
  static constexpr int STAGE_BYTES = TOKENS * PITCH * 2;
};

// Four fp32 values as two words of bf16 pairs, and their remainder x + s * w.
__device__ inline uint2 pack4(const float (&x)[4]) {
  return make_uint2(pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]));
}
__device__ inline void sub4(float (&x)[4], const uint2& w, float s) {
  x[0] = fmaf(s, bf16_lo(w.x), x[0]);
  x[1] = fmaf(s, bf16_hi(w.x), x[1]);
  x[2] = fmaf(s, bf16_lo(w.y), x[2]);
  x[3] = fmaf(s, bf16_hi(w.y), x[3]);
}

// Write one page's V block (bf16, or fp8 decoded to bf16), as loaded in lane
// order, into LDS rows 0..15; with MASK rows at or beyond `nvalid` become
// zeros.
template <int D, bool FP8, bool MASK>
__device__ inline void stage_v(const u32x4_t (&v)[Geom<D, FP8>::LOADS], int nvalid, uint16_t* vt, int lane) {
  using G = Geom<D, FP8>;
#pragma unroll
  for (int i = 0; i < G::LOADS; ++i) {
    const int e0 = (i * 64 + lane) * G::EPL;
    const int tok = e0 / D, col = e0 % D;
    u32x4_t* dst = reinterpret_cast<u32x4_t*>(vt + tok * G::PITCH + col);
    const u32x4_t zero = {0, 0, 0, 0};
    if constexpr (!FP8) {
      dst[0] = !MASK || tok < nvalid ? v[i] : zero;
    } else {
      dst[0] = !MASK || tok < nvalid ? e4m3x8_to_bf16x8(v[i].x, v[i].y) : zero;
      dst[1] = !MASK || tok < nvalid ? e4m3x8_to_bf16x8(v[i].z, v[i].w) : zero;
    }
  }
}

// Attention of up to 16 query-row columns over `npages` pages (block table
// bt, ntok tokens, at most 128 pages) of kv-head h by one wave, written as
// one partial per row. Column r16 of the wave's lanes (lane = 16 quad + r16)
// is the query row `qrow` (NULL: an unused column). COPIES = 1: its
// probabilities are rounded to bf16. COPIES > 1: each row stands in that many
// columns, 16 / COPIES lanes apart, and column `term` carries the bf16 term
// of that index of its fp32 probabilities (p = hi + mid + lo, exactly). With
// COPIES = 2, lo takes a second product on hi's column; an infinite v then
// makes elements NaN (0 times infinity), and the result false: the caller runs
// the pages AGAIN, without lo, for the elements that came out infinite or NaN
// alone (the others have all three terms). The lanes of term 0 write the row's
// partial to part_o [D] and part_lse. REUSE: the pages are read again by a
// later pass, so V too is loaded without the non-temporal hint.
template <int D, bool FP8, int COPIES, bool REUSE, bool AGAIN = false>
__device__ __forceinline__ bool attend_pages(const AttnArgs& a, int h, const int* bt, int npages, int ntok,
                                             const uint16_t* qrow, int term, float* part_o, float* part_lse,
                                             uint16_t* vt) {
  using G = Geom<D, FP8>;
  constexpr int EPL = G::EPL, LOADS = G::LOADS, PAGES = G::PAGES, DT = D / 16, PITCH = G::PITCH;
  // Probabilities that are rounded to bf16 keep the true maximum, whose own
  // probability is then exactly 1; exact ones take a lazy maximum.
  constexpr float HEADROOM = COPIES > 1 ? kLazyMax : 0.f;
  constexpr bool THIRD = COPIES == 2 && !AGAIN;  // lo's own product
  const int Hkv = a.num_kv_heads;
  const int lane = threadIdx.x & 63, r16 = lane & 15, quad = lane >> 4;
  const char* kpool = static_cast<const char*>(a.k_pages);
  const char* vpool = static_cast<const char*>(a.v_pages);

  // Every page id of the unit, two per lane, and for fp8 the pages' scales:
  // the loop reads them with v_readlane and waits for no table.
  static_assert(kRespChunkPagesMax <= 128 && kPrefixChunkPages <= 128, "two page ids per lane");
  int ids[2];
  float ksc[2] = {1.f, 1.f}, vsc[2] = {1.f, 1.f};
#pragma unroll
  for (int i = 0; i < 2; ++i) ids[i] = bt[min(64 * i + lane, npages - 1)];
  bf16x8_t qop[LOADS][EPL / 8];
#pragma unroll
  for (int j = 0; j < LOADS; ++j)
#pragma unroll
    for (int hh = 0; hh < EPL / 8; ++hh) {
      u32x4_t w = {0, 0, 0, 0};
      if (qrow != nullptr) w = *reinterpret_cast<const u32x4_t*>(qrow + (quad + 4 * j) * EPL + hh * 8);
      qop[j][hh] = __builtin_bit_cast(bf16x8_t, w);
    }
#pragma unroll
  for (int i = 0; i < 2; ++i) ids[i] = clamp_page(ids[i], a.num_pages);
  if constexpr (FP8) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      ksc[i] = a.k_scale[(size_t)ids[i] * Hkv + h];
      vsc[i] = a.v_scale[(size_t)ids[i] * Hkv + h];
    }
  }
  const auto scale_at = [&](const float (&sc)[2], int p) __attribute__((always_inline)) {
    const int q = min(p, npages - 1);
    const int x = __builtin_amdgcn_readlane(__float_as_int(sc[0]), q & 63);
    const int y = __builtin_amdgcn_readlane(__float_as_int(sc[1]), q & 63);
    return __int_as_float(q < 64 ? x : y);
  };
  // Past the last page the last page again: cache hits.
  const auto block = [&](int p) __attribute__((always_inline)) {
    const int q = min(p, npages - 1);
    const int x = __builtin_amdgcn_readlane(ids[0], q & 63), y = __builtin_amdgcn_readlane(ids[1], q & 63);
    return ((size_t)(q < 64 ? x : y) * Hkv + h) * G::BLOCK_BYTES;
  };

  // K: lane (r16, quad) holds pieces quad + 4 j of token r16's row, so its
  // elements 8 hh .. 8 hh + 7 of piece j are the A operand of product (j, hh)
  // of S^T = K Q^T (the order of head_dim inside a product is free, Q takes
  // the same one). V: 16-byte pieces in lane order, for staging. Padding rows
  // of a ragged page are read (they are inside the page) and masked when used.
  u32x4_t kx[PAGES][LOADS], vx[PAGES][LOADS];
  const uint32_t koff = (uint32_t)(r16 * G::ROW_BYTES + quad * 16), voff = (uint32_t)lane * 16;
  const auto load_k = [&](int p) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < PAGES; ++i) {
      const char* b = kpool + block(p + i);
#pragma unroll
      for (int j = 0; j < LOADS; ++j) kx[i][j] = *reinterpret_cast<const u32x4_t*>(b + koff + j * 64);
    }
  };
  const auto load_v = [&](int p) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < PAGES; ++i) {
      const char* b = vpool + block(p + i);
#pragma unroll
      for (int j = 0; j < LOADS; ++j)
        vx[i][j] = REUSE ? *reinterpret_cast<const u32x4_t*>(b + voff + j * 1024) : load_v_stream(b + voff + j * 1024);
    }
  };
  load_k(0);
  load_v(0);

  // Columns past the third term are not used.
  const float sub1 = term >= 1 ? -1.f : 0.f, sub2 = term >= 2 ? -1.f : 0.f;
  float mrow = -INFINITY, lrow = 0.f;
  f32x4_t oacc[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) oacc[dt] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  // One step from page p. `next`: request the following step's pages; the
  // last step (the only ragged one) requests nothing, since bytes read past a
  // unit's end are read again by another unit.
  const auto step = [&](int p, auto next) __attribute__((always_inline)) {
    constexpr bool NEXT = decltype(next)::value;
    const int nv = ntok - p * kPage;  // valid tokens from this step on
    // Entry (i, e): token i * 16 + quad * 4 + e of the step against column r16.
    f32x4_t sacc[PAGES];
#pragma unroll
    for (int i = 0; i < PAGES; ++i) {
      sacc[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int j = 0; j < LOADS; ++j) {
        const u32x4_t w = kx[i][j];
        if constexpr (!FP8) {
          sacc[i] = mfma16x16x32(__builtin_bit_cast(bf16x8_t, w), qop[j][0], sacc[i]);
        } else {
          sacc[i] = mfma16x16x32(__builtin_bit_cast(bf16x8_t, e4m3x8_to_bf16x8(w.x, w.y)), qop[j][0], sacc[i]);
          sacc[i] = mfma16x16x32(__builtin_bit_cast(bf16x8_t, e4m3x8_to_bf16x8(w.z, w.w)), qop[j][1], sacc[i]);
        }
      }
    }
    // Each refill stays after the last use of the registers it overwrites.
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (NEXT) load_k(p + PAGES);

    wave_lds_sync();  // the previous step's reads of the staged V are complete
#pragma unroll
    for (int i = 0; i < PAGES; ++i) stage_v<D, FP8, !NEXT>(vx[i], nv - i * kPage, vt + i * kPage * PITCH, lane);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (NEXT) load_v(p + PAGES);

#pragma unroll
    for (int i = 0; i < PAGES; ++i) {
      const float sm = FP8 ? a.qk_scale * scale_at(ksc, p + i) : a.qk_scale;
#pragma unroll
      for (int e = 0; e < 4; ++e) sacc[i][e] *= sm;
    }
    if constexpr (!NEXT) {  // padding rows may hold anything
#pragma unroll
      for (int i = 0; i < PAGES; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) sacc[i][e] = i * kPage + quad * 4 + e < nv ? sacc[i][e] : -INFINITY;
    }
    float mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < PAGES; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) mx = fmaxf(mx, sacc[i][e]);
    // Running maximum, one for the column's four quads: it moves, and the
    // accumulator is rescaled, only when some score exceeds it by more than
    // the headroom.
    if (__any(mx > mrow + HEADROOM)) {
      mx = max_xor16_32(mx);
      const float mnew = mx > mrow + HEADROOM ? mx : mrow;
      const float alpha = fast_exp2(mrow - (mnew == -INFINITY ? 0.f : mnew));
      mrow = mnew;
      lrow *= alpha;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) oacc[dt] *= alpha;
    }
    const float mu = mrow == -INFINITY ? 0.f : mrow;
    // B operand of O^T = V^T P^T: contraction slot quad*4 + e is token
    // quad*4 + e of the page, i.e. exactly this lane's four probabilities.
    bf16x4_t pop[PAGES], pop3[PAGES];
#pragma unroll
    for (int i = 0; i < PAGES; ++i) {
      float pw[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) pw[e] = fast_exp2(sacc[i][e] - mu);
      lrow += (pw[0] + pw[1]) + (pw[2] + pw[3]);
      if constexpr (FP8) {
        const float vm = scale_at(vsc, p + i);
#pragma unroll
        for (int e = 0; e < 4; ++e) pw[e] *= vm;
      }
      uint2 w = pack4(pw);
      if constexpr (COPIES >= 3) {  // a column holds what the terms before its own leave, exactly
        sub4(pw, w, sub1);
        w = pack4(pw);
        sub4(pw, w, sub2);
        w = pack4(pw);
      } else if constexpr (COPIES == 2) {
        sub4(pw, w, -1.f);
        const uint2 mid = pack4(pw);
        w = term == 0 ? w : mid;
        if constexpr (THIRD) {
          sub4(pw, mid, -1.f);
          const uint2 low = pack4(pw);
          pop3[i] = __builtin_bit_cast(bf16x4_t, term == 0 ? low : make_uint2(0, 0));
        }
      }
      pop[i] = __builtin_bit_cast(bf16x4_t, w);
    }

    wave_lds_sync();  // the staged V is visible to the whole wave
    // A operand: V^T[column dt*16 + r16][slots of quad], by transposing reads.
    const uint16_t* vtr = vt + (quad * 4 + r16 / 4) * PITCH + 4 * (r16 % 4);
    if constexpr (PAGES == 1) {
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        const bf16x4_t vo = lds_read_tr(vtr + dt * 16);
        oacc[dt] = mfma16x16x16(vo, pop[0], oacc[dt]);
        if constexpr (THIRD) oacc[dt] = mfma16x16x16(vo, pop3[0], oacc[dt]);
      }
    } else {
#pragma unroll
      for (int i = 0; i < PAGES; i += 2) {
        const bf16x8_t pp = __builtin_shufflevector(pop[i], pop[i + 1], 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
          const bf16x4_t v0 = lds_read_tr(vtr + i * kPage * PITCH + dt * 16);
          const bf16x4_t v1 = lds_read_tr(vtr + (i + 1) * kPage * PITCH + dt * 16);
          const bf16x8_t vo = __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7);
          oacc[dt] = mfma16x16x32(vo, pp, oacc[dt]);
          if constexpr (THIRD) {
            const bf16x8_t pl = __builtin_shufflevector(pop3[i], pop3[i + 1], 0, 1, 2, 3, 4, 5, 6, 7);
            oacc[dt] = mfma16x16x32(vo, pl, oacc[dt]);
          }
        }
      }
    }
  };
  int p = 0;
  for (; p + PAGES < npages; p += PAGES) step(p, std::true_type{});
  step(p, std::false_type{});

  bool done = true;
  if constexpr (THIRD) {
    bool finite = true;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int e = 0; e < 4; ++e) finite = finite && fabsf(oacc[dt][e]) < INFINITY;
    done = __all(finite);
  }

  // Add a row's terms (an infinite first term stands alone: with an infinite
  // v the others are infinite too, of either sign, or NaN), then write the
  // partial.
  const float lt = xor_sum_from<16>(lrow);
  const float inv = 1.f / lt;
  const bool store = qrow != nullptr && term == 0;
  float* dst = part_o + quad * 4;
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) {
    float v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[e] = oacc[dt][e];
      if constexpr (COPIES > 1) {
        float lo = dpp<kRowShl + 16 / COPIES>(v[e]);
        if constexpr (COPIES >= 3) lo += dpp<kRowShl + 2 * (16 / COPIES)>(v[e]);
        v[e] = fabsf(v[e]) < INFINITY ? v[e] + lo : v[e];
      }
      v[e] *= inv;
    }
    if (!store) continue;
    float4* at = reinterpret_cast<float4*>(dst + dt * 16);
    if constexpr (AGAIN) {  // this lane's own store of the first run
      const float4 first = *at;
      const float f[4] = {first.x, first.y, first.z, first.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = fabsf(f[e]) < INFINITY ? f[e] : v[e];
    }
    *at = make_float4(v[0], v[1], v[2], v[3]);
  }
  if (!AGAIN && store && quad == 0) *part_lse = (mrow + fast_log2(lt)) * kLn2;
  return done;
}

// One group-prefix unit: kv-head h of (group, chunk of prefix pages), for all
// query rows of the group's live members, 16 rows per pass. A group with more
// than 16 query rows reads the chunk again for each further pass; the chunk
// (128 KiB of K and V with 128-wide bf16 heads, half of that with 64-wide or fp8
// ones) is then mostly in this XCD's L2, its V too, which is loaded without the
// non-temporal hint then (64 rows a group, Hq 32, Hkv 4, 256 sequences: 395.9 us a
// step with the hint, 392.2 without). One pass reads its V once, as a response
// does, and takes the hint where all prefixes together (`units`, full chunks of
// every kv-head) reach 128 MiB, half of the last-level cache: less stays in that
// from step to step, and the hint gives it up. Prompts of 500-1000 tokens, responses
// of 20-200, Hkv 8, Hq 16, us without the hint and with it: 128-wide bf16, 120
// prompts of 3 sequences each (280 MiB) 123 and 106; 64-wide bf16, 200 of 3 (230
// MiB), 107 and 88; 128-wide fp8, the same, 110 and 92. Below the line, Hq 4, Hkv 2,
// 50 of 4: 128-wide bf16 25.3 without, 27.2 with; 64-wide bf16 19.3 and 20.3.
// Both forms inside one loop take 135 registers with 128-wide bf16 heads, three
// waves per SIMD; one loop each takes 126, four waves, which long batches gain 0-0.5%
// by and short groups of many passes lose 10% (8 prompts of 512-1024, 16 sequences
// each, Hq 16, Hkv 2: 71 us and 81).
template <int D, int NREP, bool FP8>
__device__ void prefix_unit(const AttnArgs& a, int item, int h, int units, uint16_t* vt) {
  const int2 it = a.view.prefix_items[item];
  const int g = clamp_group(it.x, a.num_groups);
  const int c = min(max(it.y, 0), a.view.max_prefix_chunks - 1);
  const int P = clamp_len(a.prefix_lens[g], a.max_prefix_pages);
  const int ntok = min(kPrefixChunkPages * kPage, P - c * (kPrefixChunkPages * kPage));
  if (ntok <= 0) return;
  const int moff = a.view.grp_off[g];
  const int R = (a.view.grp_off[g + 1] - moff) * NREP;
  const int* bt = a.prefix_block_table + (size_t)g * a.max_prefix_pages + c * kPrefixChunkPages;
  constexpr int kStreamUnits = (128 << 20) / (kPrefixChunkPages * 2 * Geom<D, FP8>::BLOCK_BYTES);
  const int r16 = threadIdx.x & 15;
  for (int r0 = 0; r0 < R; r0 += 16) {
    const int rr = r0 + r16;
    const uint16_t* qrow = nullptr;
    int part = 0;
    if (rr < R) {
      const int mem = rr / NREP, rep = rr - mem * NREP;
      const int sq = min(max(a.view.grp_members[moff + mem], 0), a.num_seqs - 1);
      const int rowid = sq * a.num_q_heads + h * NREP + rep;
      qrow = static_cast<const uint16_t*>(a.q) + (size_t)rowid * D;
      part = clamp_part(rowid * a.view.parts_per_row + c, a.view.max_parts);
    }
    float *po = a.view.part_o + (size_t)part * D, *pl = a.view.part_lse + part;
    const int npages = cdiv(ntok, kPage);
    if (R <= 16 && units >= kStreamUnits) {
      attend_pages<D, FP8, 1, false>(a, h, bt, npages, ntok, qrow, 0, po, pl, vt);
      return;
    }
    attend_pages<D, FP8, 1, true>(a, h, bt, npages, ntok, qrow, 0, po, pl, vt);
  }
}

// The NREP query rows of sequence s and kv-head h over the ntok > 0 tokens of
// block table bt; columns are copies r16 / NREP of query row r16 % NREP, and
// part_o, part_lse the lane's row's.
template <int D, int NREP, bool FP8>
__device__ __forceinline__ void attend_rows(const AttnArgs& a, int s, int h, const int* bt, int ntok, float* part_o,
                                            float* part_lse, uint16_t* vt) {
  const int r16 = threadIdx.x & 15;
  const uint16_t* qrow =
      static_cast<const uint16_t*>(a.q) + ((size_t)s * a.num_q_heads + h * NREP + r16 % NREP) * D;
  const int npages = cdiv(ntok, kPage);
  const bool done =
      attend_pages<D, FP8, 16 / NREP, false>(a, h, bt, npages, ntok, qrow, r16 / NREP, part_o, part_lse, vt);
  if constexpr (NREP == 8) {
    if (!done)
      attend_pages<D, FP8, 2, false, true>(a, h, bt, npages, ntok, qrow, r16 / NREP, part_o, part_lse, vt);
  }
}

// One response unit: kv-head h of response item `item`.
template <int D, int NREP, bool FP8>
__device__ void resp_unit(const AttnArgs& a, int item, int h, uint16_t* vt) {
  // The item record: sequence, first page index in its block table, tokens, slot.
  const int4 m = a.view.resp_items[item];
  const int s = min(max(m.x, 0), a.num_seqs - 1);
  const int p0 = min(max(m.y, 0), a.max_resp_pages);
  const int ntok = min(max(m.z, 0), min(kRespChunkPagesMax, a.max_resp_pages - p0) * kPage);
  const int slot = min(max(m.w, 0), a.view.parts_per_row - 1);
  if (ntok == 0) return;
  const int* bt = a.resp_block_table + (size_t)s * a.max_resp_pages + p0;
  const int rowid = s * a.num_q_heads + h * NREP + (threadIdx.x & 15) % NREP;
  const int part = clamp_part(rowid * a.view.parts_per_row + slot, a.view.max_parts);
  attend_rows<D, NREP, FP8>(a, s, h, bt, ntok, a.view.part_o + (size_t)part * D, a.view.part_lse + part, vt);
}

// All partial results in one launch, one unit per workgroup: the first
// blocks take the group-prefix units (dispatched first; their short,
// latency-bound MFMA work overlaps the response units that fill the rest of
// the GPU), the following blocks the response units in plan order (big items
// first, then small ones by decreasing size), and blocks beyond the planned
// counts exit at once. Unit kinds are not interleaved by block id: workgroups
// are dealt round-robin to XCDs and then to shader engines, and any periodic
// pattern of unit kinds would correlate with that and unbalance them. The
// counts are clamped to the plan's capacity, so even a workspace that was
// never planned cannot send a wave outside the item lists.
template <int D, int NREP, bool FP8>
__global__ __launch_bounds__(64)
void attn_parts_kernel(const AttnArgs a) {
  __shared__ __attribute__((aligned(16))) uint16_t vt[Geom<D, FP8>::STAGE_BYTES / 2];
  const int Hkv = a.num_kv_heads;
  const int n_pre = min(max(a.view.hdr[kHdrPrefixItems], 0), a.view.max_prefix_items) * Hkv;
  const int n_resp = min(max(a.view.hdr[kHdrRespItems], 0), a.view.max_resp_items) * Hkv;
  const int b = blockIdx.x;
  if (b < n_pre) {
    const int item = b / Hkv;
    prefix_unit<D, NREP, FP8>(a, item, b - item * Hkv, n_pre, vt);
    return;
  }
  const int resp = b - n_pre;
  if (resp < n_resp) {
    int item = resp / Hkv, h = resp - item * Hkv;
    if constexpr (FP8) {
      // Workgroups are dealt to the 8 XCDs in turn, so eight items interleaved
      // put all kv-heads of an item on one XCD: the scales of a page's heads
      // share a cache line, which its L2 then fetches once (256 sequences of
      // 8192-32768 tokens: 1677 -> 1662 us a step, d 64 905 -> 887). bf16
      // pools have no such line and are 0.1-0.5% slower this way.
      const int row = resp / (8 * Hkv), k = resp - row * (8 * Hkv);
      if ((row + 1) * (8 * Hkv) <= n_resp) {
        item = row * 8 + k % 8;
        h = k / 8;
      }
    }
    resp_unit<D, NREP, FP8>(a, item, h, vt);
  }
}

// A small batch whole, in one launch: a workgroup per (sequence, kv-head)
// splits the prefix and the response pages into at most kSmallWaves pieces, a
// wave each, and merges their partials in LDS; each sequence reads its
// group's prefix for itself. Both kinds of pages load V with the hint: prefix
// pages without it are 1-7% faster where one large group shares a long prefix
// (64 sequences of 900 + 200 tokens, 2 kv-heads: 17.4 -> 16.6 us), and 1-4%
// slower where several groups of 16 have as much response (4 x 16 of 300 + 300,
// 4 kv-heads 13.6 -> 14.0). Block 0 makes the batch's plan, as the three-launch
// form leaves it in the workspace, and a row's merged result becomes its first
// partial there (the others empty), so that a combine on the workspace gives out
// and lse again. Bound by the chain of round trips and steps of one wave (4
// sequences of 192 tokens, 2 kv-heads: 8.2 us a call, three launches 13.2; the
// partials are 0.1 us of it).
template <int D, int NREP, bool FP8>
__global__ __launch_bounds__(64 * kSmallWaves) void attn_small_kernel(const AttnArgs a, const PlanArgs p, uint16_t* out,
                                                                      float* lse_out) {
  constexpr int kStage = Geom<D, FP8>::STAGE_BYTES / 2;
  struct Work {
    uint16_t vt[kSmallWaves][kStage];
    float o[kSmallWaves][NREP][D];
    float lse[kSmallWaves][NREP];
  };
  __shared__ __attribute__((aligned(16))) union Smem {
    Work w;
    int cnt[kPlanMaxGroups];
    __device__ Smem() {}
  } sm;
  if (blockIdx.x == 0) {
    if (threadIdx.x < 64) plan_small(p, sm.cnt);
    return;
  }
  const int Hkv = a.num_kv_heads;
  const int s = (int)(blockIdx.x - 1) / Hkv, h = (int)(blockIdx.x - 1) - s * Hkv;
  const int t = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int g = clamp_group(a.seq_to_group[s], a.num_groups);
  const int L = clamp_len(a.resp_lens[s], a.max_resp_pages), P = clamp_len(a.prefix_lens[g], a.max_prefix_pages);
  // Pieces of `per` pages, of the prefix first: cdiv(x, per) + cdiv(y, per) is
  // at most kSmallWaves for x + y <= (kSmallWaves - 1) per.
  const int np = cdiv(P, kPage), nr = cdiv(L, kPage), step = Geom<D, FP8>::PAGES;
  const int per = cdiv(max(cdiv(np + nr, kSmallWaves - 1), 1), step) * step;
  const int pre = cdiv(np, per), parts = pre + cdiv(nr, per);
  if (wave < parts) {
    const bool in_prefix = wave < pre;
    const int p0 = (in_prefix ? wave : wave - pre) * per;
    const int ntok = min(per * kPage, (in_prefix ? P : L) - p0 * kPage);
    const int* bt = in_prefix ? a.prefix_block_table + (size_t)g * a.max_prefix_pages
                              : a.resp_block_table + (size_t)s * a.max_resp_pages;
    const int rep = (t & 15) % NREP;
    attend_rows<D, NREP, FP8>(a, s, h, bt + p0, ntok, sm.w.o[wave][rep], &sm.w.lse[wave][rep], sm.w.vt[wave]);
  }
  __syncthreads();
  for (int i = t; i < NREP * D / 2; i += 64 * kSmallWaves) {
    const int rep = i / (D / 2), col = i % (D / 2) * 2;
    float mx = -INFINITY;
    for (int k = 0; k < parts; ++k) mx = fmaxf(mx, sm.w.lse[k][rep]);
    float x = 0.f, y = 0.f, wsum = 0.f;
    for (int k = 0; k < parts && mx != -INFINITY; ++k) {
      const float l = sm.w.lse[k][rep];
      if (l == -INFINITY) continue;  // an empty part, as the combine reads it
      const float w = fast_exp2((l - mx) * kLog2e);
      wsum += w;
      x = fmaf(w, sm.w.o[k][rep][col], x);
      y = fmaf(w, sm.w.o[k][rep][col + 1], y);
    }
    const float inv = wsum > 0.f ? 1.f / wsum : 0.f;
    const size_t row = (size_t)s * a.num_q_heads + h * NREP + rep;
    x *= inv;
    y *= inv;
    const float lse = wsum > 0.f ? mx + fast_log2(wsum) * kLn2 : -INFINITY;
    *reinterpret_cast<uint32_t*>(out + row * D + col) = pack_bf16x2(x, y);
    if (lse_out != nullptr && col == 0) lse_out[row] = lse;
    const int slots = a.view.parts_per_row;
    if (slots == 0) continue;  // tables without pages: no partials
    const size_t part = row * slots;
    *reinterpret_cast<float2*>(a.view.part_o + part * D + col) = make_float2(x, y);
    // The combine gives NaN and an lse of minus infinity, as here, for a part
    // of lse plus infinity.
    if (col == 0) a.view.part_lse[part] = wsum != wsum ? INFINITY : lse;
    for (int k = 1 + col / 2; k < slots; k += D / 2) a.view.part_lse[part + k] = -INFINITY;
  }
}

template <int D, bool FP8>
hipError_t small_by_nrep(const AttnArgs& a, const PlanArgs& p, int n_rep, uint16_t* out, float* lse, hipStream_t st) {
  const dim3 grid((unsigned)(a.num_seqs * a.num_kv_heads + 1)), block(64 * kSmallWaves);
  switch (n_rep) {
    case 1: attn_small_kernel<D, 1, FP8><<<grid, block, 0, st>>>(a, p, out, lse); break;
    case 2: attn_small_kernel<D, 2, FP8><<<grid, block, 0, st>>>(a, p, out, lse); break;
    case 4: attn_small_kernel<D, 4, FP8><<<grid, block, 0, st>>>(a, p, out, lse); break;
    case 8: attn_small_kernel<D, 8, FP8><<<grid, block, 0, st>>>(a, p, out, lse); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// Grid: one block per unit of the largest plan that fits the workspace.
template <int D, int NREP, bool FP8>
hipError_t launch_one(const AttnArgs& a, long long prefix_blocks, long long resp_blocks, hipStream_t st) {
  const long long blocks = prefix_blocks + resp_blocks;
  attn_parts_kernel<D, NREP, FP8><<<dim3((unsigned)blocks), dim3(64), 0, st>>>(a);
  return hipGetLastError();
}

template <int D, bool FP8>
hipError_t by_nrep(const AttnArgs& a, int n_rep, long long pb, long long rb, hipStream_t st) {
  switch (n_rep) {
    case 1: return launch_one<D, 1, FP8>(a, pb, rb, st);
    case 2: return launch_one<D, 2, FP8>(a, pb, rb, st);
    case 4: return launch_one<D, 4, FP8>(a, pb, rb, st);
    case 8: return launch_one<D, 8, FP8>(a, pb, rb, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_attn_small(const AttnArgs& a, const PlanArgs& p, int head_dim, int n_rep, bool fp8, void* out,
                             float* lse, hipStream_t stream) {
  if (a.num_seqs <= 0) return hipSuccess;
  if (a.num_seqs > kSmallPlanMaxSeqs || p.num_seqs != a.num_seqs) return hipErrorInvalidValue;
  uint16_t* o = static_cast<uint16_t*>(out);
  if (head_dim == 128) return fp8 ? small_by_nrep<128, true>(a, p, n_rep, o, lse, stream) : small_by_nrep<128, false>(a, p, n_rep, o, lse, stream);
  if (head_dim == 64) return fp8 ? small_by_nrep<64, true>(a, p, n_rep, o, lse, stream) : small_by_nrep<64, false>(a, p, n_rep, o, lse, stream);
  return hipErrorInvalidValue;
}

hipError_t launch_attn_parts(const AttnArgs& a, int head_dim, int n_rep, bool fp8, long long max_prefix_items,
                             long long max_resp_items, hipStream_t stream) {
  const long long pb = max_prefix_items * a.num_kv_heads, rb = max_resp_items * a.num_kv_heads;
  if (pb + rb <= 0) return hipSuccess;
  if (head_dim == 128) return fp8 ? by_nrep<128, true>(a, n_rep, pb, rb, stream) : by_nrep<128, false>(a, n_rep, pb, rb, stream);
  if (head_dim == 64) return fp8 ? by_nrep<64, true>(a, n_rep, pb, rb, stream) : by_nrep<64, false>(a, n_rep, pb, rb, stream);
  return hipErrorInvalidValue;
}

}  // namespace rp
