// KV append: the new token of sequence s goes into response slot L =
// resp_lens[s] (page resp_block_table[s][L / 16], row L % 16). bf16 pools copy
// the values, 16 bytes per thread; fp8 pools apply the per-(page, kv-head)
// scale rule of append_fp8_row, D / 4 lanes per row, K and V of a kv-head side
// by side in one wave.
#include "rp_device.h"
#include "rp_internal.h"

#pragma clang fp contract(off)

namespace rp {
namespace {

constexpr int kAppendThreads = 256;

template <int D>
__global__ __launch_bounds__(kAppendThreads) void append_bf16_kernel(const AppendArgs a) {
  constexpr int CPR = D / 8;  // 16-byte pieces per row
  const int per_seq = 2 * a.num_kv_heads * CPR;
  const long long i = (long long)blockIdx.x * kAppendThreads + threadIdx.x;
  const int s = (int)(i / per_seq);
  if (s >= a.num_seqs) return;
  const int c = (int)(i - (long long)s * per_seq);
  const int h = c / (2 * CPR), v = c / CPR % 2, col = c % CPR * 8;
  const int L = a.resp_lens[s];
  const uint16_t* src = static_cast<const uint16_t*>(v ? a.v_new : a.k_new);
  const uint4 w = *reinterpret_cast<const uint4*>(src + ((size_t)s * a.num_kv_heads + h) * D + col);
  if (L < 0 || L >= a.max_resp_pages * kPage) return;  // no slot for the new token
  const int page = clamp_page(a.resp_block_table[(size_t)s * a.max_resp_pages + L / kPage], a.num_pages);
  uint16_t* dst = static_cast<uint16_t*>(v ? a.v_pages : a.k_pages);
  *reinterpret_cast<uint4*>(dst + (((size_t)page * a.num_kv_heads + h) * kPage + L % kPage) * D + col) = w;
}

template <int D>
__global__ __launch_bounds__(64) void append_fp8_kernel(const AppendArgs a) {
  constexpr int G = D / 4;  // lanes per row
  const int Hkv = a.num_kv_heads;
  const int s = blockIdx.x / Hkv, h = blockIdx.x - s * Hkv;
  const int L = a.resp_lens[s];
  if (L < 0 || L >= a.max_resp_pages * kPage) return;  // no slot for the new token
  const int lane = threadIdx.x, v = lane / G & 1, l = lane % G;
  const uint16_t* src = static_cast<const uint16_t*>(v ? a.v_new : a.k_new) + ((size_t)s * Hkv + h) * D;
  const uint2 w = *reinterpret_cast<const uint2*>(src + l * 4);
  const int page = clamp_page(a.resp_block_table[(size_t)s * a.max_resp_pages + L / kPage], a.num_pages);
  const size_t slot = (size_t)page * Hkv + h;
  float* scale = (v ? a.v_scale : a.k_scale) + slot;
  const float x[4] = {bf16_lo(w.x), bf16_hi(w.x), bf16_lo(w.y), bf16_hi(w.y)};
  const int col[1] = {l * 4};
  RequantJob job = {};
  if (lane < 2 * G)
    job = append_fp8_row<D, G, 4>(static_cast<uint8_t*>(v ? a.v_pages : a.k_pages) + slot * (kPage * D), scale, *scale,
                                  L % kPage, x, col, l == 0);
  requantise_fp8_rows<D>(job, l == 0, lane);
}

// Layout checker (test utility): records the number of bad entries and one example.
__device__ void report(int* res, int kind, int index, int value) {
  if (atomicAdd(&res[0], 1) == 0) {
    res[1] = kind;
    res[2] = index;
    res[3] = value;
  }
}

__global__ __launch_bounds__(256) void validate_kernel(const ValidateArgs a) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  const int nt = gridDim.x * blockDim.x;
  for (int s = t; s < a.num_seqs; s += nt) {
    const int g = a.seq_to_group[s];
    if (g < 0 || g >= a.num_groups) report(a.result, 1, s, g);
    const int L = a.resp_lens[s];
    if (L < 0 || L > a.max_resp_pages * kPage) {
      report(a.result, 3, s, L);
      continue;
    }
    for (int p = 0; p < cdiv(L, kPage); ++p) {
      const int page = a.resp_block_table[(size_t)s * a.max_resp_pages + p];
      if (page < 0 || page >= a.num_pages) report(a.result, 5, s, page);
    }
  }
  for (int g = t; g < a.num_groups; g += nt) {
    const int P = a.prefix_lens[g];
    if (P < 0 || P > a.max_prefix_pages * kPage) {
      report(a.result, 2, g, P);
      continue;
    }
    for (int p = 0; p < cdiv(P, kPage); ++p) {
      const int page = a.prefix_block_table[(size_t)g * a.max_prefix_pages + p];
      if (page < 0 || page >= a.num_pages) report(a.result, 4, g, page);
    }
  }
}

}  // namespace

hipError_t launch_append(const AppendArgs& a, int head_dim, bool fp8, hipStream_t stream) {
  const long long rows = (long long)a.num_seqs * a.num_kv_heads;
  if (rows <= 0) return hipSuccess;
  if (head_dim != 128 && head_dim != 64) return hipErrorInvalidValue;
  if (fp8) {
    const dim3 grid((unsigned)rows), block(64);
    if (head_dim == 128) append_fp8_kernel<128><<<grid, block, 0, stream>>>(a);
    else append_fp8_kernel<64><<<grid, block, 0, stream>>>(a);
  } else {
    const dim3 grid((unsigned)((rows * 2 * (head_dim / 8) + kAppendThreads - 1) / kAppendThreads)), block(kAppendThreads);
    if (head_dim == 128) append_bf16_kernel<128><<<grid, block, 0, stream>>>(a);
    else append_bf16_kernel<64><<<grid, block, 0, stream>>>(a);
  }
  return hipGetLastError();
}

hipError_t launch_validate(const ValidateArgs& a, hipStream_t stream) {
  validate_kernel<<<64, 256, 0, stream>>>(a);
  return hipGetLastError();
}

}  // namespace rp
