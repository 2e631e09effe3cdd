// fp32 replay kernels for any head_dim <= 256 and any GQA group; head dimensions
// that are multiples of 4 up to 128 run on the matrix cores instead
// (fwd_f32_mfma.hip, bwd_f32_mfma.hip), but for the backward of a few keys
// or rows (f32_dq_small, f32_dkdv_small).  One wave owns one (query row, head) --
// or, for the response-key gradients, one (key, KV head) -- and walks its keys
// one at a time with an online softmax; lane l holds channels l, l+64, l+128,
// l+192.
#include "f32_rows.h"

namespace ls {
namespace {
using namespace f32r;

constexpr int kPer = 4;  // channels per lane (256 / 64)

// Eq. qwen-local-attn for one split.
__global__ __launch_bounds__(256) void fwd_f32_kernel(FwdArgs a) {
  const int lane = threadIdx.x & 63;
  const int64_t pair = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);  // row * Hq + head
  if (pair >= (int64_t)a.n_q * a.n_q_heads) return;
  const int row = (int)(pair / a.n_q_heads), head = (int)(pair - (int64_t)row * a.n_q_heads);
  fwd_row<kPer>(a, blockIdx.z, row, head, lane);
}

// dq over the keys of [kv_begin, kv_end) visible to the row: scale * sum dS k.
__global__ __launch_bounds__(256) void bwd_dq_f32_kernel(BwdArgs a) {
  const int lane = threadIdx.x & 63;
  const int64_t pair = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (pair >= (int64_t)a.n_q * a.n_q_heads) return;
  const int row = (int)(pair / a.n_q_heads), head = (int)(pair - (int64_t)row * a.n_q_heads);
  float acc[kPer];
  dq_row<kPer>(a, a.kv_begin, min(a.kv_end, a.q_pos0 + row + 1), row, head, lane, acc);
  float* dq = a.dq + pair * a.head_dim;
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int d = lane + k * 64;
    if (d < a.head_dim) dq[d] = a.accumulate_dq ? dq[d] + a.scale * acc[k] : a.scale * acc[k];
  }
}

// Gradients of one response key j >= prefix_len of KV head g, summed over
// every (row, head of the group) that sees it (dk times scale).
__global__ __launch_bounds__(256) void bwd_dkdv_f32_kernel(BwdArgs a, int64_t key0, int64_t n_keys) {
  const int lane = threadIdx.x & 63;
  const int64_t item = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);  // key * Hkv + g
  if (item >= n_keys * a.n_kv_heads) return;
  const int64_t jj = item / a.n_kv_heads;
  const int g = (int)(item - jj * a.n_kv_heads);
  const int64_t j = key0 + jj;
  float dk[kPer], dv[kPer];
  dkdv_key<kPer>(a, j, g, 0, (int64_t)a.n_q * a.group, lane, dk, dv);
  const int64_t r = (j - a.prefix_len) * a.n_kv_heads + g;
  float* dkr = a.dk_resp + r * a.head_dim;
  float* dvr = a.dv_resp + r * a.head_dim_v;
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int d = lane + k * 64;
    if (d < a.head_dim) dkr[d] = a.accumulate_dkv ? dkr[d] + a.scale * dk[k] : a.scale * dk[k];
    if (d < a.head_dim_v) dvr[d] = a.accumulate_dkv ? dvr[d] + dv[k] : dv[k];
  }
}

}  // namespace

hipError_t launch_fwd_f32(const FwdArgs& a, hipStream_t stream) {
  if (f32_mfma_fits(a.head_dim, a.head_dim_v, a.n_kv_heads)) return launch_fwd_f32_mfma(a, stream);
  const unsigned blocks = (unsigned)(((int64_t)a.n_q * a.n_q_heads + 3) / 4);
  hipLaunchKernelGGL(fwd_f32_kernel, dim3(blocks, 1, a.n_splits), dim3(256), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_dq_f32_generic(const BwdArgs& a, hipStream_t stream) {
  const unsigned blocks = (unsigned)(((int64_t)a.n_q * a.n_q_heads + 3) / 4);
  hipLaunchKernelGGL(bwd_dq_f32_kernel, dim3(blocks), dim3(256), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_dkdv_f32_generic(const BwdArgs& a, int64_t key0, hipStream_t stream) {
  const int64_t n_keys = a.kv_end - key0;
  const unsigned blocks = (unsigned)((n_keys * a.n_kv_heads + 3) / 4);
  hipLaunchKernelGGL(bwd_dkdv_f32_kernel, dim3(blocks), dim3(256), 0, stream, a, key0, n_keys);
  return hipGetLastError();
}

}  // namespace ls
