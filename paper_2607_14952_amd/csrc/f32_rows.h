// fp32 attention one key (or one query row) at a time by one wave: lane l holds
// channels l, l + 64, .. (kPer of them).  The generic kernels work this way, and
// the matrix-core kernels where a result is not finite: a tile's product adds 0
// times the values of keys that a row does not see, which is NaN for an infinity
// or NaN among them, so such a row is formed again from the keys that it sees.
#pragma once
#include <math.h>

#include "ls_internal.h"

namespace ls {
namespace f32r {

__device__ __forceinline__ float wave_sum(float x) {
  for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off);
  return x;
}

__device__ __forceinline__ int64_t phys_row(const int32_t* __restrict__ table, int64_t j,
                                            int log2_page) {
  const int64_t S = int64_t(1) << log2_page;
  return (int64_t)table[j >> log2_page] * S + (j & (S - 1));
}

// This lane's channels of a row of d floats (0 past its end).
template <int kPer>
__device__ __forceinline__ void load_channels(float* v, const float* row, int d, int lane) {
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int c = lane + k * 64;
    v[k] = c < d ? row[c] : 0.f;
  }
}

// Eq. qwen-local-attn of (row, head) over split sp: normalized output and
// natural-log normalizer.
template <int kPer>
__device__ __forceinline__ void fwd_row(const FwdArgs& a, int sp, int row, int head, int lane) {
  const int g = head / a.group;   // any group size, not only powers of two
  const int64_t pair = (int64_t)row * a.n_q_heads + head;
  const int64_t kb = a.split_begin(sp);
  const int64_t ke = min(a.split_end(sp), a.q_pos0 + row + 1);
  const float* kp = static_cast<const float*>(a.k_pool);
  const float* vp = static_cast<const float*>(a.v_pool);
  float qv[kPer], o[kPer];
  load_channels<kPer>(qv, static_cast<const float*>(a.q) + pair * a.head_dim, a.head_dim, lane);
#pragma unroll
  for (int k = 0; k < kPer; ++k) o[k] = 0.f;
  float m = -INFINITY, l = 0.f;
  for (int64_t j = kb; j < ke; ++j) {
    const int64_t pr = phys_row(a.page_table, j, a.log2_page);
    const float* kr = kp + pr * a.k_pos_stride + (int64_t)g * a.head_dim;
    const float* vr = vp + pr * a.v_pos_stride + (int64_t)g * a.head_dim_v;
    float part = 0.f;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int d = lane + k * 64;
      if (d < a.head_dim) part = fmaf(qv[k], kr[d], part);
    }
    const float s2 = wave_sum(part) * a.scale_log2;
    const float m_new = fmaxf(m, s2);
    const float alpha = __builtin_amdgcn_exp2f(m - m_new);
    const float p = __builtin_amdgcn_exp2f(s2 - m_new);
    l = fmaf(l, alpha, p);
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int d = lane + k * 64;
      o[k] = fmaf(o[k], alpha, d < a.head_dim_v ? p * vr[d] : 0.f);
    }
    m = m_new;
  }
  float* out = a.out_part + ((int64_t)sp * a.n_q * a.n_q_heads + pair) * a.head_dim_v;
  const float inv = l > 0.f ? 1.f / l : 0.f;
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int d = lane + k * 64;
    if (d < a.head_dim_v) out[d] = o[k] * inv;
  }
  if (lane == 0)
    a.lse_part[(int64_t)sp * a.n_q * a.n_q_heads + (int64_t)head * a.n_q + row] =
        l > 0.f ? (m + __builtin_amdgcn_logf(l)) * kLn2 : -INFINITY;
}

// sum dS k of (row, head) over the keys of [kb, ke), all visible to it:
// P = exp(s - lse), dS = P (dO . v - Delta).
template <int kPer>
__device__ __forceinline__ void dq_row(const BwdArgs& a, int64_t kb, int64_t ke, int row, int head,
                                       int lane, float* acc) {
  const int g = head / a.group;   // any group size, not only powers of two
  const int64_t pair = (int64_t)row * a.n_q_heads + head;
  const float* kp = static_cast<const float*>(a.k_pool);
  const float* vp = static_cast<const float*>(a.v_pool);
  const float lse2 = a.lse2[(int64_t)head * a.n_q + row];
  const float delta = a.delta[(int64_t)head * a.n_q + row];
  float qv[kPer], dov[kPer];
  load_channels<kPer>(qv, static_cast<const float*>(a.q) + pair * a.head_dim, a.head_dim, lane);
  load_channels<kPer>(dov, static_cast<const float*>(a.d_out) + pair * a.head_dim_v, a.head_dim_v,
                      lane);
#pragma unroll
  for (int k = 0; k < kPer; ++k) acc[k] = 0.f;
  for (int64_t j = kb; j < ke; ++j) {
    const int64_t pr = phys_row(a.page_table, j, a.log2_page);
    const float* kr = kp + pr * a.k_pos_stride + (int64_t)g * a.head_dim;
    const float* vr = vp + pr * a.v_pos_stride + (int64_t)g * a.head_dim_v;
    float ps = 0.f, pd = 0.f;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int d = lane + k * 64;
      if (d < a.head_dim) ps = fmaf(qv[k], kr[d], ps);
      if (d < a.head_dim_v) pd = fmaf(dov[k], vr[d], pd);
    }
    const float s2 = wave_sum(ps) * a.scale_log2;
    const float dp = wave_sum(pd);
    const float p = __builtin_amdgcn_exp2f(s2 - lse2);
    const float ds = p * (dp - delta);
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int d = lane + k * 64;
      if (d < a.head_dim) acc[k] = fmaf(ds, kr[d], acc[k]);
    }
  }
}

// Gradients of key j of KV head g, summed over the packed rows of [row_lo, row_hi)
// that see it (packed row r: token r / group, head r % group of the KV head's):
// dv = sum P dO, dk = sum dS q.
template <int kPer>
__device__ __forceinline__ void dkdv_key(const BwdArgs& a, int64_t j, int g, int64_t row_lo,
                                         int64_t row_hi, int lane, float* dk, float* dv) {
  const int64_t pr = phys_row(a.page_table, j, a.log2_page);
  float kv[kPer], vv[kPer];
  load_channels<kPer>(kv, static_cast<const float*>(a.k_pool) + pr * a.k_pos_stride +
                              (int64_t)g * a.head_dim, a.head_dim, lane);
  load_channels<kPer>(vv, static_cast<const float*>(a.v_pool) + pr * a.v_pos_stride +
                              (int64_t)g * a.head_dim_v, a.head_dim_v, lane);
#pragma unroll
  for (int k = 0; k < kPer; ++k) dk[k] = dv[k] = 0.f;
  const int64_t first = j > a.q_pos0 ? (j - a.q_pos0) * a.group : 0;
  int64_t r = max(row_lo, first), row = r / a.group;
  int hh = (int)(r - row * a.group);
  for (; r < row_hi; ++r) {
    const int head = g * a.group + hh;
    const int64_t pair = row * a.n_q_heads + head;
    float qv[kPer], dov[kPer];
    load_channels<kPer>(qv, static_cast<const float*>(a.q) + pair * a.head_dim, a.head_dim, lane);
    load_channels<kPer>(dov, static_cast<const float*>(a.d_out) + pair * a.head_dim_v,
                        a.head_dim_v, lane);
    float ps = 0.f, pd = 0.f;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      ps = fmaf(qv[k], kv[k], ps);
      pd = fmaf(dov[k], vv[k], pd);
    }
    const int64_t o = (int64_t)head * a.n_q + row;
    const float p = __builtin_amdgcn_exp2f(wave_sum(ps) * a.scale_log2 - a.lse2[o]);
    const float ds = p * (wave_sum(pd) - a.delta[o]);
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      dk[k] = fmaf(ds, qv[k], dk[k]);
      dv[k] = fmaf(p, dov[k], dv[k]);
    }
    if (++hh == a.group) {
      hh = 0;
      ++row;
    }
  }
}

}  // namespace f32r
}  // namespace ls
