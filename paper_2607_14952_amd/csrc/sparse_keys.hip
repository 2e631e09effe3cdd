// Sparse latent replay: resolution of each token's key list (selected prefix
// positions, then the response window) to physical latent rows, once per call;
// the forward and the backward both stream their tiles from it.
#include "sparse_common.h"

namespace ls {
namespace {
using namespace sparse;

// ---------------------------------------------------------------- key lists
// One workgroup per token t: phys[t][k] for k < n_max is the physical latent
// row of key k of the token's list, which holds the selected prefix positions
// that lie inside [0, prefix_len) in their given order (an entry outside the
// prefix, such as the -1 pad of a selection shorter than k, selects no key),
// then the response window prefix_len .. q_pos0 + t.  ntok[t] is the list's
// length; entries past it repeat its last key so tile loads stay inside the
// pool (the tile kernels mask keys at or past ntok[t]).
// kU entries of each thread are in flight at a time (8: 2,048 of the list; 2 for
// lists of up to 512, where more would only be idle lanes' work): the
// walk is a chain of dependent loads (entry, page, store), so what counts is how
// few times it is entered (2,048 selections, 24 tokens: 8.0 -> 4.9 us).
template <int kU>
__global__ __launch_bounds__(256) void sparse_phys_kernel(SparseArgs a) {
  __shared__ int wave_total[kU][4];
  const int t = (int)blockIdx.x, tid = (int)threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int32_t* sel = a.idx + (int64_t)t * a.topk;
  int32_t* out = a.phys + (int64_t)t * a.n_max;
  int base = 0;   // valid selections written so far (uniform)
  for (int k0 = 0; k0 < a.topk; k0 += 256 * kU) {
    int32_t pos[kU];
    int before[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int k = k0 + 256 * u + tid;
      pos[u] = k < a.topk ? sel[k] : -1;
    }
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      if ((int64_t)pos[u] >= a.prefix_len) pos[u] = -1;
      const uint64_t ball = __ballot(pos[u] >= 0);
      before[u] = __popcll(ball & ((uint64_t(1) << lane) - 1));
      if (lane == 0) wave_total[u][w] = __popcll(ball);
    }
    __syncthreads();
    int32_t page[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) page[u] = a.page_table[(pos[u] < 0 ? 0 : pos[u]) >> a.log2_page];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      int off = base + before[u];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        off += v < w ? wave_total[u][v] : 0;
        base += wave_total[u][v];
      }
      if (pos[u] >= 0)
        out[off] = (page[u] << a.log2_page) | (pos[u] & ((1 << a.log2_page) - 1));
    }
    __syncthreads();
  }
  const int n_t = base + (int)a.window0 + t + 1;
  for (int k0 = base; k0 < a.n_max; k0 += 256 * kU) {
    int32_t row[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int k = min(k0 + 256 * u + tid, n_t - 1);
      row[u] = (int32_t)phys_pos(a.page_table, a.prefix_len + k - base, a.log2_page);
    }
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int k = k0 + 256 * u + tid;
      if (k < a.n_max) out[k] = row[u];
    }
  }
  if (tid == 0) a.ntok[t] = n_t;
}

}  // namespace

hipError_t launch_sparse_phys(const SparseArgs& a, hipStream_t stream) {
  if (a.n_max <= 512)
    hipLaunchKernelGGL(sparse_phys_kernel<2>, dim3((unsigned)a.n_q), dim3(256), 0, stream, a);
  else
    hipLaunchKernelGGL(sparse_phys_kernel<8>, dim3((unsigned)a.n_q), dim3(256), 0, stream, a);
  return hipGetLastError();
}

}  // namespace ls
