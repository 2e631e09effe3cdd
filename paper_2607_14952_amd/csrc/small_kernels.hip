// Bandwidth-bound kernels of the replay path: the page-table gather, the
// log-sum-exp merge of split results, and the backward row statistics; and a
// read-only streaming probe that measures the HBM read ceiling.
#include <math.h>

#include <algorithm>

#include "ls_internal.h"

namespace ls {
namespace {

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;

// ---------------------------------------------------------------- gather
// Logical position j lives in physical page page_table[j >> log2_page] at
// slot j & (S - 1); each position row is copied in 16-byte units.
__global__ __launch_bounds__(256) void gather_kernel(const char* __restrict__ k_pool,
                                                     const char* __restrict__ v_pool,
                                                     const int32_t* __restrict__ page_table,
                                                     int64_t pos_begin, int64_t n, int log2_page,
                                                     int64_t k_row_bytes, int64_t v_row_bytes,
                                                     char* __restrict__ k_out,
                                                     char* __restrict__ v_out) {
  const bool is_v = blockIdx.y == 1;
  const char* pool = is_v ? v_pool : k_pool;
  char* dst = is_v ? v_out : k_out;
  const int64_t row_bytes = is_v ? v_row_bytes : k_row_bytes;
  const int64_t units = row_bytes >> 4;
  const int64_t total = n * units;
  const int64_t S = int64_t(1) << log2_page;
  for (int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; u < total;
       u += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = u / units, c = u - r * units;
    const int64_t j = pos_begin + r;
    const int64_t page = page_table[j >> log2_page];
    const int64_t phys_row = page * S + (j & (S - 1));
    const u32x4 v = *reinterpret_cast<const u32x4*>(pool + phys_row * row_bytes + c * 16);
    *reinterpret_cast<u32x4*>(dst + r * row_bytes + c * 16) = v;
  }
}

// Inverse of the gather: dense rows -> their logical positions in the pool.
__global__ __launch_bounds__(256) void scatter_kernel(char* __restrict__ k_pool,
                                                      char* __restrict__ v_pool,
                                                      const int32_t* __restrict__ page_table,
                                                      int64_t pos_begin, int64_t n, int log2_page,
                                                      int64_t k_row_bytes, int64_t v_row_bytes,
                                                      const char* __restrict__ k_src,
                                                      const char* __restrict__ v_src) {
  const bool is_v = blockIdx.y == 1;
  char* pool = is_v ? v_pool : k_pool;
  const char* src = is_v ? v_src : k_src;
  const int64_t row_bytes = is_v ? v_row_bytes : k_row_bytes;
  const int64_t units = row_bytes >> 4;
  const int64_t total = n * units;
  const int64_t S = int64_t(1) << log2_page;
  for (int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; u < total;
       u += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = u / units, c = u - r * units;
    const int64_t j = pos_begin + r;
    const int64_t page = page_table[j >> log2_page];
    const int64_t phys_row = page * S + (j & (S - 1));
    *reinterpret_cast<u32x4*>(pool + phys_row * row_bytes + c * 16) =
        *reinterpret_cast<const u32x4*>(src + r * row_bytes + c * 16);
  }
}

// ---------------------------------------------------------------- merge
// Eq. qwen-lse-parts: m = max l_r, a = sum e^(l_r - m), n = sum e^(l_r - m) o_r;
// o = n / a, l = m + log a (computed with exp2/log2 and converted to natural
// log), over each group of parts and, with several groups, once more over the
// groups' results in group order.
// BF16_NUM (the last level only): the production composition described after
// Eq. qwen-global-attn, n reduced in bf16: each term e^(l_r - m) o_r is rounded
// to bf16 and added in part order with the running sum rounded to bf16 after
// every addition (m, a and l stay fp32).
//
// An item is 4 output values of one (row, head).  Two kernels, both bound by
// reading the parts once: the wide one gives an item one thread, the narrow one
// sixteen waves of a workgroup that share its parts, for calls too small to
// fill the chip with threads (launch_merge).
__device__ __forceinline__ float round_bf16(float x) { return (float)(__bf16)x; }

constexpr int kMU = 8;   // parts read at a time, so that their loads are in flight together

struct MergeArgs {
  const float* out_part;
  const float* lse_part;
  float* group_out;         // [n_groups, rows, dv] and [n_groups, heads, n_q]; null with one group
  float* group_lse;
  void* out;
  float* lse;
  int32_t n_q, n_heads, dv4, n_groups;
  int32_t begin[kMaxMergeGroups], end[kMaxMergeGroups];   // parts of each group
  int32_t per;              // narrow kernel: parts per unit
};

struct MergeItem {
  int64_t t, rows, lse_off;   // item index, rows * heads, offset into an lse array
  int d4;
  __device__ __forceinline__ MergeItem(const MergeArgs& a, int64_t item) : t(item) {
    rows = (int64_t)a.n_q * a.n_heads;
    const int64_t rh = t / a.dv4;               // row-major (row, head)
    d4 = (int)(t - rh * a.dv4);
    const int row = (int)(rh / a.n_heads), head = (int)(rh - (int64_t)row * a.n_heads);
    lse_off = (int64_t)head * a.n_q + row;
  }
};

__device__ __forceinline__ float merged_lse(float m, float a) {
  return m == -INFINITY ? -INFINITY : m + __builtin_amdgcn_logf(a) * kLn2;
}

template <bool BF16_NUM>
__device__ __forceinline__ void add_part(float l, const f32x4& o, float m2, float& a, f32x4& acc) {
  const float w = __builtin_amdgcn_exp2f(fmaf(l, kLog2e, -m2));   // 0 for l = -inf
  a += w;
  if (BF16_NUM) {
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] = round_bf16(acc[e] + round_bf16(w * o[e]));
  } else {
    acc += w * o;
  }
}

// Weighted sum over parts [p0, p1) of arrays out [., rows * dv] and lse
// [., rows]: m, a and acc as above (acc = a = 0 where every part is empty).
template <bool BF16_NUM>
__device__ __forceinline__ void merge_parts(const float* out, const float* lse, int p0, int p1,
                                            int dv4, const MergeItem& it, float& m, float& a,
                                            f32x4& acc) {
  const f32x4* src = reinterpret_cast<const f32x4*>(out) + it.t;
  m = -INFINITY;
  acc = f32x4{0.f, 0.f, 0.f, 0.f};
  a = 0.f;
  if (p1 - p0 <= kMU) {   // one batch: log-normalizers and values load together
    float l[kMU];
    f32x4 o[kMU];
#pragma unroll
    for (int u = 0; u < kMU; ++u) {
      l[u] = -INFINITY;
      if (p0 + u < p1) {
        l[u] = lse[(int64_t)(p0 + u) * it.rows + it.lse_off];
        o[u] = src[(int64_t)(p0 + u) * it.rows * dv4];
      }
    }
#pragma unroll
    for (int u = 0; u < kMU; ++u) m = fmaxf(m, l[u]);
    if (m == -INFINITY) return;
#pragma unroll
    for (int u = 0; u < kMU; ++u) {
      if (p0 + u < p1) add_part<BF16_NUM>(l[u], o[u], m * kLog2e, a, acc);
    }
    return;
  }
  // whole batches without a test per part, which would compute their addresses anew
  // each time (98 parts of 120 rows of 128, one thread each: 19.2 us, so 12.3), then
  // the rest, which reads its last part again in place of missing ones
  const int64_t l_step = it.rows, o_step = it.rows * dv4;
  const float* lp = lse + (int64_t)p0 * l_step + it.lse_off;
  int left = p1 - p0;
  for (; left >= kMU; left -= kMU, lp += kMU * l_step) {
    float l[kMU];
#pragma unroll
    for (int u = 0; u < kMU; ++u) l[u] = lp[u * l_step];
#pragma unroll
    for (int u = 0; u < kMU; ++u) m = fmaxf(m, l[u]);
  }
  if (left > 0) {
    float l[kMU];
#pragma unroll
    for (int u = 0; u < kMU; ++u) l[u] = lp[min(u, left - 1) * l_step];
#pragma unroll
    for (int u = 0; u < kMU; ++u) m = fmaxf(m, l[u]);
  }
  if (m == -INFINITY) return;
  const float m2 = m * kLog2e;
  lp = lse + (int64_t)p0 * l_step + it.lse_off;
  src += (int64_t)p0 * o_step;
  left = p1 - p0;
  for (; left >= kMU; left -= kMU, lp += kMU * l_step, src += kMU * o_step) {
    float l[kMU];
    f32x4 o[kMU];
#pragma unroll
    for (int u = 0; u < kMU; ++u) {
      l[u] = lp[u * l_step];
      o[u] = src[u * o_step];
    }
#pragma unroll
    for (int u = 0; u < kMU; ++u) add_part<BF16_NUM>(l[u], o[u], m2, a, acc);
  }
  if (left > 0) {
    float l[kMU];
    f32x4 o[kMU];
#pragma unroll
    for (int u = 0; u < kMU; ++u) {
      l[u] = lp[min(u, left - 1) * l_step];
      o[u] = src[min(u, left - 1) * o_step];
    }
#pragma unroll
    for (int u = 0; u < kMU; ++u)
      if (u < left) add_part<BF16_NUM>(l[u], o[u], m2, a, acc);
  }
}

template <bool OUT_BF16>
__device__ __forceinline__ void store_item(void* out, int64_t t, const f32x4& v) {
  if (OUT_BF16) {
    bf16x4 r;
    r[0] = (__bf16)v[0]; r[1] = (__bf16)v[1]; r[2] = (__bf16)v[2]; r[3] = (__bf16)v[3];
    reinterpret_cast<bf16x4*>(out)[t] = r;
  } else {
    reinterpret_cast<f32x4*>(out)[t] = v;
  }
}

// One thread per item.  With kGroups the groups' results go to group_out /
// group_lse, from where the thread reads its own values again for the last level.
template <bool OUT_BF16, bool BF16_NUM, bool kGroups>
__global__ __launch_bounds__(256) void merge_kernel(MergeArgs g) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const MergeItem it(g, t);
  if (t >= it.rows * g.dv4) return;
  float m, a;
  f32x4 acc;
  if constexpr (kGroups) {
    for (int k = 0; k < g.n_groups; ++k) {
      merge_parts<false>(g.out_part, g.lse_part, g.begin[k], g.end[k], g.dv4, it, m, a, acc);
      if (m != -INFINITY) acc *= 1.0f / a;
      reinterpret_cast<f32x4*>(g.group_out)[(int64_t)k * it.rows * g.dv4 + t] = acc;
      // (every thread of the row writes the same value, which it reads back)
      g.group_lse[(int64_t)k * it.rows + it.lse_off] = merged_lse(m, a);
    }
    merge_parts<BF16_NUM>(g.group_out, g.group_lse, 0, g.n_groups, g.dv4, it, m, a, acc);
  } else {
    merge_parts<BF16_NUM>(g.out_part, g.lse_part, g.begin[0], g.end[0], g.dv4, it, m, a, acc);
  }
  if (m != -INFINITY) acc *= 1.0f / a;
  store_item<OUT_BF16>(g.out, t, acc);
  if (it.d4 == 0) g.lse[it.lse_off] = merged_lse(m, a);
}

// 64 items per workgroup of 16 waves.  The groups' parts are cut into units of
// at most `per` parts (no more than kMergeUnits in all); waves take units in
// turn and leave their sums in LDS, then take groups, then wave 0 composes
// these.
constexpr int kMergeUnits = 64;
template <bool OUT_BF16, bool BF16_NUM>
__global__ __launch_bounds__(1024) void merge_narrow_kernel(MergeArgs g) {
  __shared__ f32x4 s_acc[kMergeUnits][64];
  __shared__ float s_m[kMergeUnits][64], s_a[kMergeUnits][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t t = (int64_t)blockIdx.x * 64 + lane;
  const int64_t last = (int64_t)g.n_q * g.n_heads * g.dv4 - 1;
  const MergeItem it(g, min(t, last));
  float m, a;
  f32x4 acc;
  // units are numbered group by group: lane k holds group k's parts and units
  const int gk = min(lane, g.n_groups - 1);
  const int g_begin = g.begin[gk], g_end = g.end[gk];
  const int g_units = lane < g.n_groups ? (g_end - g_begin + g.per - 1) / g.per : 0;
  int g_last = g_units;   // one past the group's last unit
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int o = __shfl_up(g_last, d);
    if (lane >= d) g_last += o;
  }
  const int g_first = g_last - g_units;
  const int n_units = __builtin_amdgcn_readlane(g_last, 63);
  for (int u = w; u < n_units; u += 16) {
    const int k = __popcll(__ballot(g_last <= u));
    const int p = __builtin_amdgcn_readlane(g_begin, k) +
                  (u - __builtin_amdgcn_readlane(g_first, k)) * g.per;
    merge_parts<false>(g.out_part, g.lse_part, p,
                       min(p + g.per, __builtin_amdgcn_readlane(g_end, k)), g.dv4, it, m, a, acc);
    s_acc[u][lane] = acc;
    s_m[u][lane] = m;
    s_a[u][lane] = a;
  }
  __syncthreads();
  // group k's result replaces its first unit (only the group's wave reads its units)
  for (int k = w; k < g.n_groups; k += 16) {
    const int u0 = __builtin_amdgcn_readlane(g_first, k), u1 = __builtin_amdgcn_readlane(g_last, k);
    m = -INFINITY;
    for (int v = u0; v < u1; ++v) m = fmaxf(m, s_m[v][lane]);
    acc = f32x4{0.f, 0.f, 0.f, 0.f};
    a = 0.f;
    if (m != -INFINITY) {
      for (int v = u0; v < u1; ++v) {
        const float x = __builtin_amdgcn_exp2f((s_m[v][lane] - m) * kLog2e);
        a = fmaf(x, s_a[v][lane], a);
        acc += x * s_acc[v][lane];
      }
      acc *= 1.0f / a;
    }
    const float l = merged_lse(m, a);
    if (g.n_groups == 1) {
      if (t <= last) {
        store_item<OUT_BF16>(g.out, t, acc);
        if (it.d4 == 0) g.lse[it.lse_off] = l;
      }
    } else {
      s_acc[u0][lane] = acc;
      s_m[u0][lane] = l;
      if (t <= last) {
        reinterpret_cast<f32x4*>(g.group_out)[(int64_t)k * it.rows * g.dv4 + t] = acc;
        if (it.d4 == 0) g.group_lse[(int64_t)k * it.rows + it.lse_off] = l;
      }
    }
  }
  if (g.n_groups == 1) return;
  __syncthreads();
  if (w > 0) return;
  m = -INFINITY;
  for (int k = 0; k < g.n_groups; ++k)
    m = fmaxf(m, s_m[__builtin_amdgcn_readlane(g_first, k)][lane]);
  acc = f32x4{0.f, 0.f, 0.f, 0.f};
  a = 0.f;
  if (m != -INFINITY) {
    for (int k = 0; k < g.n_groups; ++k) {
      const int u = __builtin_amdgcn_readlane(g_first, k);
      const float x = __builtin_amdgcn_exp2f((s_m[u][lane] - m) * kLog2e);
      a += x;
      const f32x4 o = s_acc[u][lane];
      if (BF16_NUM) {
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] = round_bf16(acc[e] + round_bf16(x * o[e]));
      } else {
        acc += x * o;
      }
    }
    acc *= 1.0f / a;
  }
  if (t > last) return;
  store_item<OUT_BF16>(g.out, t, acc);
  if (it.d4 == 0) g.lse[it.lse_off] = merged_lse(m, a);
}

// ---------------------------------------------------------------- bwd prep
// One wave per (row, head): Delta = d_out . out, and the log-normalizer in
// base 2 (rows without any visible key get +inf so that P = 0).
template <typename TD, typename TO>
__global__ __launch_bounds__(256) void prep_kernel(const TD* __restrict__ d_out,
                                                   const TO* __restrict__ out,
                                                   const float* __restrict__ lse, int n_q,
                                                   int n_heads, int dv, float* __restrict__ delta,
                                                   float* __restrict__ lse2) {
  const int64_t rh = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (rh >= (int64_t)n_q * n_heads) return;
  const int row = (int)(rh / n_heads), head = (int)(rh - (int64_t)row * n_heads);
  float acc = 0.f;
  for (int d = lane; d < dv; d += 64)
    acc += (float)d_out[rh * dv + d] * (float)out[rh * dv + d];
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
  if (lane == 0) {
    const int64_t o = (int64_t)head * n_q + row;
    delta[o] = acc;
    const float l = lse[o];
    lse2[o] = (l == -INFINITY) ? INFINITY : l * kLog2e;
  }
}

// The same with dv = 64 kE: lane l takes elements kE l .. kE l + kE - 1 of the
// row, one vector load of each operand, so a wave reads each row in one
// coalesced instruction instead of kE narrow ones.
template <typename T, int kE>
__device__ __forceinline__ void load_as_float(const T* __restrict__ p, float* f) {
  typedef __attribute__((__vector_size__(kE * sizeof(T)))) T V;
  const V v = *reinterpret_cast<const V*>(p);
#pragma unroll
  for (int e = 0; e < kE; ++e) f[e] = (float)v[e];
}

template <typename TD, typename TO, int kE>
__global__ __launch_bounds__(256) void prep_vec_kernel(const TD* __restrict__ d_out,
                                                       const TO* __restrict__ out,
                                                       const float* __restrict__ lse, int n_q,
                                                       int n_heads, float* __restrict__ delta,
                                                       float* __restrict__ lse2) {
  constexpr int kDv = 64 * kE;
  const int64_t rh = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (rh >= (int64_t)n_q * n_heads) return;
  const int row = (int)(rh / n_heads), head = (int)(rh - (int64_t)row * n_heads);
  float d[kE], o[kE];
  load_as_float<TD, kE>(d_out + rh * kDv + kE * lane, d);
  load_as_float<TO, kE>(out + rh * kDv + kE * lane, o);
  float acc = 0.f;
#pragma unroll
  for (int e = 0; e < kE; ++e) acc = fmaf(d[e], o[e], acc);
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
  if (lane == 0) {
    const int64_t i = (int64_t)head * n_q + row;
    delta[i] = acc;
    const float l = lse[i];
    lse2[i] = (l == -INFINITY) ? INFINITY : l * kLog2e;
  }
}

// ---------------------------------------------------------------- dq chunks
// dq (+)= scale * the sum of each key range's partials part[z0 .. z1) [., n4],
// range by range: what a launch per range would leave, to the bit (the choice of
// the kernel and the order of a range's sum depend on n4 and its own chunks
// only).  An item is 4 values; eight chunks' loads are in flight.
__device__ __forceinline__ f32x4 sum_chunks(const f32x4* part, int64_t n4, int64_t i, int c, int end) {
  constexpr int kU = 8;
  f32x4 sum = {0.f, 0.f, 0.f, 0.f};
  for (; c + kU <= end; c += kU) {
    f32x4 v[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) v[u] = part[(int64_t)(c + u) * n4 + i];
#pragma unroll
    for (int u = 0; u < kU; ++u) sum += v[u];
  }
  for (; c < end; ++c) sum += part[(int64_t)c * n4 + i];
  return sum;
}

// out (the value so far, when there is one) += scale * sum, with one rounding
__device__ __forceinline__ void add_range(f32x4& out, bool some, const f32x4& sum, float scale) {
  if (!some) {
    out = sum * scale;
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) out[e] = fmaf(sum[e], scale, out[e]);
  }
}

// One thread per item.
__global__ __launch_bounds__(256) void dq_reduce_kernel(const f32x4* __restrict__ part,
                                                        DqRanges r, int64_t n4, float scale,
                                                        int accumulate, f32x4* __restrict__ dq) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n4) return;
  f32x4 out = {0.f, 0.f, 0.f, 0.f};
  if (accumulate) out = dq[i];
  for (int k = 0; k < r.n; ++k)
    add_range(out, k > 0 || accumulate, sum_chunks(part, n4, i, r.z0[k], r.z0[k + 1]), scale);
  dq[i] = out;
}

// Few items and many chunks (1 row: 128 chunks for 1,024 items, a chain of 32
// loads for one thread): 64 items per workgroup, whose 16 waves each sum a
// sixteenth of a range's chunks (backward of 16 rows x 8 ranges of 32,768 keys:
// 330 -> 264 us).
__global__ __launch_bounds__(1024) void dq_reduce_narrow_kernel(const f32x4* __restrict__ part,
                                                                DqRanges r, int64_t n4,
                                                                float scale, int accumulate,
                                                                f32x4* __restrict__ dq) {
  __shared__ f32x4 sums[16][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t i = min((int64_t)blockIdx.x * 64 + lane, n4 - 1);
  f32x4 out = {0.f, 0.f, 0.f, 0.f};
  if (accumulate) out = dq[i];
  for (int k = 0; k < r.n; ++k) {
    const int z = r.z0[k], n = r.z0[k + 1] - z;
    sums[w][lane] = sum_chunks(part, n4, i, z + n * w / 16, z + n * (w + 1) / 16);
    __syncthreads();
    if (w == 0) {
      f32x4 sum = sums[0][lane];
#pragma unroll
      for (int v = 1; v < 16; ++v) sum += sums[v][lane];
      add_range(out, k > 0 || accumulate, sum, scale);
    }
    __syncthreads();
  }
  if (w == 0 && (int64_t)blockIdx.x * 64 + lane < n4) dq[i] = out;
}

// ---------------------------------------------------------------- HBM read probe
// Reads n16 16-byte units once and XORs their 32-bit words: a read-only
// streaming pass with no arithmetic to speak of, the measured read ceiling the
// bandwidth-bound kernels are compared with.  Each thread keeps 8 loads of 16
// bytes in flight; a wave's XOR goes to *out with one atomic.
__global__ __launch_bounds__(256) void hbm_read_kernel(const u32x4* __restrict__ buf,
                                                       int64_t n16, uint32_t* __restrict__ out) {
  constexpr int kU = 8;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  uint32_t x = 0;
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (; i + (kU - 1) * stride < n16; i += kU * stride) {
    u32x4 v[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) v[u] = __builtin_nontemporal_load(buf + i + u * stride);
#pragma unroll
    for (int u = 0; u < kU; ++u) x ^= v[u][0] ^ v[u][1] ^ v[u][2] ^ v[u][3];
  }
  for (; i < n16; i += stride) {
    const u32x4 v = buf[i];
    x ^= v[0] ^ v[1] ^ v[2] ^ v[3];
  }
  for (int off = 32; off > 0; off >>= 1) x ^= (uint32_t)__shfl_xor((int)x, off);
  if ((threadIdx.x & 63) == 0) atomicXor(out, x);
}

}  // namespace

hipError_t launch_gather(const void* k_pool, const void* v_pool, const int32_t* page_table,
                         int64_t pos_begin, int64_t pos_end, int log2_page, int64_t k_row_elems,
                         int64_t v_row_elems, int esize, void* k_out, void* v_out,
                         hipStream_t stream) {
  const int64_t n = pos_end - pos_begin;
  const int64_t units = n * ((k_row_elems > v_row_elems ? k_row_elems : v_row_elems) * esize / 16);
  int64_t blocks = (units + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(gather_kernel, dim3((unsigned)blocks, 2), dim3(256), 0, stream,
                     (const char*)k_pool, (const char*)v_pool, page_table, pos_begin, n, log2_page,
                     k_row_elems * esize, v_row_elems * esize, (char*)k_out, (char*)v_out);
  return hipGetLastError();
}

hipError_t launch_scatter(void* k_pool, void* v_pool, const int32_t* page_table,
                          int64_t pos_begin, int64_t pos_end, int log2_page, int64_t k_row_elems,
                          int64_t v_row_elems, int esize, const void* k_src, const void* v_src,
                          hipStream_t stream) {
  const int64_t n = pos_end - pos_begin;
  const int64_t units = n * ((k_row_elems > v_row_elems ? k_row_elems : v_row_elems) * esize / 16);
  int64_t blocks = (units + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(scatter_kernel, dim3((unsigned)blocks, 2), dim3(256), 0, stream,
                     (char*)k_pool, (char*)v_pool, page_table, pos_begin, n, log2_page,
                     k_row_elems * esize, v_row_elems * esize, (const char*)k_src,
                     (const char*)v_src);
  return hipGetLastError();
}

hipError_t launch_merge(const float* out_part, const float* lse_part, const int32_t* begin,
                        const int32_t* end, int n_groups, int n_q, int n_heads, int dv,
                        bool out_bf16, bool bf16_numerator, float* group_out, float* group_lse,
                        void* out, float* lse, hipStream_t stream) {
  MergeArgs g = {};
  g.out_part = out_part;
  g.lse_part = lse_part;
  g.group_out = group_out;
  g.group_lse = group_lse;
  g.out = out;
  g.lse = lse;
  g.n_q = n_q;
  g.n_heads = n_heads;
  g.dv4 = dv / 4;
  g.n_groups = n_groups;
  int most = 0;
  for (int k = 0; k < n_groups; ++k) {
    g.begin[k] = begin[k];
    g.end[k] = end[k];
    most = std::max(most, end[k] - begin[k]);
  }
  const int64_t items = (int64_t)n_q * n_heads * g.dv4;
  // The narrow kernel: where one thread per item leaves under two waves per
  // SIMD and the parts are more than one batch of loads (16 rows x 16 heads,
  // 257 parts in 9 groups: 79 us in ten launches of one thread per item, 17 us
  // here; 1 row, 65 parts: 37 us in ten launches, 7 us here with 129 parts).  A
  // single group's bf16 numerator is added in part order, which one thread does.
  const bool narrow = items <= 512 * 64 && (most > kMU || n_groups > 1) &&
                      !(bf16_numerator && n_groups == 1);
  if (narrow) {
    auto units = [&](int per) {
      int n = 0;
      for (int k = 0; k < n_groups; ++k) n += (end[k] - begin[k] + per - 1) / per;
      return n;
    };
    g.per = kMU;
    while (units(g.per) > kMergeUnits) g.per += kMU;   // (n_groups <= kMergeUnits)
  }
#define LS_MERGE(OB, BN)                                                                       \
  if (narrow)                                                                                  \
    hipLaunchKernelGGL((merge_narrow_kernel<OB, BN>), dim3((unsigned)((items + 63) / 64)),     \
                       dim3(1024), 0, stream, g);                                              \
  else if (n_groups > 1)                                                                       \
    hipLaunchKernelGGL((merge_kernel<OB, BN, true>), dim3((unsigned)((items + 255) / 256)),    \
                       dim3(256), 0, stream, g);                                               \
  else                                                                                         \
    hipLaunchKernelGGL((merge_kernel<OB, BN, false>), dim3((unsigned)((items + 255) / 256)),   \
                       dim3(256), 0, stream, g)
  if (out_bf16 && bf16_numerator) {
    LS_MERGE(true, true);
  } else if (out_bf16) {
    LS_MERGE(true, false);
  } else if (bf16_numerator) {
    LS_MERGE(false, true);
  } else {
    LS_MERGE(false, false);
  }
#undef LS_MERGE
  return hipGetLastError();
}

hipError_t launch_bwd_prep(const void* d_out, const void* out, bool dout_bf16, bool out_bf16,
                           const float* lse, int n_q, int n_heads, int dv, float* delta,
                           float* lse2, hipStream_t stream) {
  const unsigned blocks = (unsigned)(((int64_t)n_q * n_heads + 3) / 4);
  // whole rows of dv = 256 or 512 with 16-byte aligned bases take the vector
  // loads (row starts are then aligned for both element sizes)
  const bool vec = (dv == 256 || dv == 512) &&
                   (((uintptr_t)d_out | (uintptr_t)out) & 15) == 0;
#define LS_PREP(TD, TO)                                                                       \
  if (vec && dv == 512)                                                                       \
    hipLaunchKernelGGL((prep_vec_kernel<TD, TO, 8>), dim3(blocks), dim3(256), 0, stream,      \
                       (const TD*)d_out, (const TO*)out, lse, n_q, n_heads, delta, lse2);     \
  else if (vec)                                                                               \
    hipLaunchKernelGGL((prep_vec_kernel<TD, TO, 4>), dim3(blocks), dim3(256), 0, stream,      \
                       (const TD*)d_out, (const TO*)out, lse, n_q, n_heads, delta, lse2);     \
  else                                                                                        \
    hipLaunchKernelGGL((prep_kernel<TD, TO>), dim3(blocks), dim3(256), 0, stream,             \
                       (const TD*)d_out, (const TO*)out, lse, n_q, n_heads, dv, delta, lse2)
  if (dout_bf16 && out_bf16) {
    LS_PREP(__bf16, __bf16);
  } else if (dout_bf16) {
    LS_PREP(__bf16, float);
  } else if (out_bf16) {
    LS_PREP(float, __bf16);
  } else {
    LS_PREP(float, float);
  }
#undef LS_PREP
  return hipGetLastError();
}

hipError_t launch_dq_reduce(const float* part, const DqRanges& r, int64_t n, float scale,
                            bool accumulate, float* dq, hipStream_t stream) {
  const int64_t n4 = n / 4;
  if (n4 <= 32768)   // under two waves of one-thread items per SIMD
    hipLaunchKernelGGL(dq_reduce_narrow_kernel, dim3((unsigned)((n4 + 63) / 64)), dim3(1024), 0,
                       stream, (const f32x4*)part, r, n4, scale, accumulate ? 1 : 0, (f32x4*)dq);
  else
    hipLaunchKernelGGL(dq_reduce_kernel, dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, stream,
                       (const f32x4*)part, r, n4, scale, accumulate ? 1 : 0, (f32x4*)dq);
  return hipGetLastError();
}

hipError_t launch_hbm_read(const void* buf, int64_t n16, uint32_t* out, hipStream_t stream) {
  hipLaunchKernelGGL(hbm_read_kernel, dim3(2048), dim3(256), 0, stream, (const u32x4*)buf, n16,
                     out);
  return hipGetLastError();
}

}  // namespace ls
