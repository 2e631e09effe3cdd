// fp32 split-KV forward on the matrix cores (f32_mfma.h) for head dimensions
// that are multiples of 4 up to 128, any GQA group (Eq. qwen-local-attn): products
// and sums in fp32 as the generic kernel forms them, but a 32-key x 32-row score
// tile per MFMA chain.
//
// A workgroup is 4 waves = kRW groups of 32 packed query rows of one KV head
// (packed row r is token r / G, head g*G + r % G) x 4 / kRW key slots: per
// iteration the whole workgroup stages 4 / kRW consecutive 32-key tiles of K
// and V in LDS, and each wave forms, for its rows and its slot's tile,
//   S^T (32 keys x its 32 rows) = K Q^T        kDP/2 MFMAs of K = 2,
//   O^T (kDP x 32 rows) += V^T P^T             16 * kDP/32 MFMAs of K = 2.
// With kRW = 1 the waves' partial softmaxes are merged through LDS at the end.
//
// The MFMA bounds it (64 cycles each; one 16-byte LDS read per 4 of them), so
// what matters is that every SIMD has a wave: calls whose 128-row workgroups
// leave CUs idle take kRW = 1, four times as many workgroups with a quarter of the
// keys per wave, where these finish sooner (f32_fwd_wide).
#include "f32_mfma.h"

namespace ls {
namespace {
using namespace f32m;

template <int kDP, int kRW>
__global__ __launch_bounds__(256, kRW == 4 ? 2 : 1) void fwd_f32_mfma_kernel(FwdArgs a) {
  constexpr int kKW = 4 / kRW;                // key slots
  constexpr int kKS = kRowS<kDP>, kVS = kColS<kDP>;
  constexpr int kDB = kDP / 32;               // output dimension blocks
  __shared__ __attribute__((aligned(16))) float smem[kKW * 32 * (kKS + kVS)];
  float* const ks = smem;
  float* const vs = smem + kKW * 32 * kKS;

  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int rw = w % kRW, kw = w / kRW;
  const int j = lane & 31, h = lane >> 5;
  const int g = blockIdx.y, sp = blockIdx.z;
  const int G = a.group, D = a.head_dim, Dv = a.head_dim_v;
  const int64_t rows_total = (int64_t)a.n_q * G;
  const int64_t row0 = (int64_t)blockIdx.x * (32 * kRW);
  const int64_t prow = row0 + rw * 32 + j;
  const bool row_ok = prow < rows_total;
  const int tok = (int)(prow / G);
  const int head = g * G + (int)(prow - (int64_t)tok * G);
  const int64_t kb = a.split_begin(sp), ke = a.split_end(sp);
  const int tok_last = (int)(min(rows_total, row0 + 32 * kRW) - 1) / G;
  const int64_t k_hi = min(ke, a.q_pos0 + tok_last + 1);            // keys of the workgroup
  const int64_t my_lim = row_ok ? min(ke, a.q_pos0 + tok + 1) : kb;  // this row: [kb, my_lim)
  // below: visible to every row (of a whole row group)
  const int64_t k_all =
      row0 + 32 * kRW <= rows_total ? min(ke, a.q_pos0 + (int)(row0 / G) + 1) : kb;
  const int64_t k_lo = kb & ~int64_t(31);
  const int n_tiles = k_hi > kb ? (int)((k_hi - k_lo + 31) / 32) : 0;

  float qv[kDP / 2];
  const int64_t rh = row_ok ? (int64_t)tok * a.n_q_heads + head : 0;   // (rows past the end: row 0)
  load_half_row<kDP>(qv, static_cast<const float*>(a.q) + rh * D, D, h);
  f32x16 oacc[kDB];
#pragma unroll
  for (int b = 0; b < kDB; ++b) oacc[b] = zero16();
  float m_run = -INFINITY, l_run = 0.f;

  KvStage<kDP, kKW> stage;
  if (n_tiles > 0) {
    stage.load_pages(a, k_lo, kb, k_hi, tid);
    stage.load(a, g, k_lo, kb, k_hi, tid);
  }
  for (int t = 0; t < n_tiles; t += kKW) {
    const int64_t t0 = k_lo + (int64_t)t * 32;
    __syncthreads();   // every wave is done with the previous tiles
    stage.template store<kKS, kVS>(a, ks, vs, tid);
    __syncthreads();
    if (t + kKW < n_tiles) stage.load(a, g, t0 + 32 * kKW, kb, k_hi, tid);
    if (t + kw >= n_tiles) continue;   // (uniform per wave; the barriers above are not skipped)

    const int64_t tw = t0 + 32 * kw;
    f32x16 s = row_product<kDP, kKS>(ks + kw * 32 * kKS, qv, j, h);
    if (tw < kb || tw + 32 > k_all) {
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (!in_rows(r, h, kb - tw, my_lim - tw)) s[r] = -INFINITY;
    }
    float mx = s[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
    mx = half_max(mx) * a.scale_log2;
    const float m_new = fmaxf(m_run, mx);
    const float m_use = m_new == -INFINITY ? 0.f : m_new;
    const float alpha = __builtin_amdgcn_exp2f(m_run - m_use);
    float psum = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      s[r] = __builtin_amdgcn_exp2f(fmaf(s[r], a.scale_log2, -m_use));
      psum += s[r];
    }
    l_run = fmaf(l_run, alpha, psum);
    m_run = m_new;
#pragma unroll
    for (int b = 0; b < kDB; ++b) oacc[b] *= alpha;
    col_product<kDP, kVS>(vs + kw * 32 * kVS, s, oacc, j, h);
  }

  float l_tot = half_sum(l_run);
  if constexpr (kKW > 1) {
    // merge the key slots: slot 0's wave adds the others' accumulators, each
    // rescaled to the common maximum, in slot order
    constexpr int kAcc = kDB * 16 * 64;
    static_assert((kKW - 1) * kAcc + 2 * kKW * 64 <= kKW * 32 * (kKS + kVS), "merge area");
    __syncthreads();
    float* stat = smem + (kKW - 1) * kAcc;
    stat[(2 * kw) * 64 + lane] = m_run;
    stat[(2 * kw + 1) * 64 + lane] = l_tot;
    if (kw > 0) acc_to_lds<kDB>(smem + (kw - 1) * kAcc, oacc, lane);
    __syncthreads();
    if (kw > 0) return;
    float m = m_run;
#pragma unroll
    for (int k = 1; k < kKW; ++k) m = fmaxf(m, stat[2 * k * 64 + lane]);
    const float m_use = m == -INFINITY ? 0.f : m;
    const float w0 = __builtin_amdgcn_exp2f(m_run - m_use);
    l_tot *= w0;
#pragma unroll
    for (int b = 0; b < kDB; ++b) oacc[b] *= w0;
#pragma unroll
    for (int k = 1; k < kKW; ++k) {
      const float wk = __builtin_amdgcn_exp2f(stat[2 * k * 64 + lane] - m_use);
      l_tot = fmaf(wk, stat[(2 * k + 1) * 64 + lane], l_tot);
      acc_add_lds<kDB>(oacc, smem + (k - 1) * kAcc, wk, lane);
    }
    m_run = m;
  }
  if (row_ok) {
    float* out = a.out_part + (((int64_t)sp * a.n_q + tok) * a.n_q_heads + head) * Dv;
    const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
#pragma unroll
    for (int b = 0; b < kDB; ++b) {
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const int d = 32 * b + 8 * q4 + 4 * h;
        f32x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = oacc[b][4 * q4 + e] * inv;
        if (d < Dv) *reinterpret_cast<f32x4*>(out + d) = v;
      }
    }
    if (h == 0)
      a.lse_part[((int64_t)sp * a.n_q_heads + head) * a.n_q + tok] =
          l_tot > 0.f ? (m_run + __builtin_amdgcn_logf(l_tot)) * kLn2 : -INFINITY;
  }
  // rows to form again key by key (f32_rows.h); the rows past the end are none
  uint32_t again = not_finite<kDB>(oacc) & (uint32_t)__ballot(row_ok);
  if (__builtin_expect(again != 0, 0)) {
    __threadfence();   // (the values stored so far come first)
    for (; again; again &= again - 1) {
      const int i = __builtin_ctz(again);
      f32r::fwd_row<2>(a, opaque(blockIdx.z), __builtin_amdgcn_readlane(tok, i),
                       __builtin_amdgcn_readlane(head, i), lane_id());
    }
  }
}

template <int kDP>
void launch(const FwdArgs& a, hipStream_t stream) {
  const int64_t rows = (int64_t)a.n_q * a.group;
  if (f32_fwd_wide(a)) {
    const dim3 grid((unsigned)((rows + 127) / 128), a.n_kv_heads, a.n_splits);
    hipLaunchKernelGGL((fwd_f32_mfma_kernel<kDP, 4>), grid, dim3(256), 0, stream, a);
  } else {
    const dim3 grid((unsigned)((rows + 31) / 32), a.n_kv_heads, a.n_splits);
    hipLaunchKernelGGL((fwd_f32_mfma_kernel<kDP, 1>), grid, dim3(256), 0, stream, a);
  }
}

}  // namespace

bool f32_mfma_fits(int head_dim, int head_dim_v, int n_kv_heads) {
  return head_dim <= kMaxWidth && head_dim_v <= kMaxWidth && head_dim % 4 == 0 &&
         head_dim_v % 4 == 0 && n_kv_heads <= 65535;   // (a grid dimension)
}

hipError_t launch_fwd_f32_mfma(const FwdArgs& a, hipStream_t stream) {
  const int d = a.head_dim > a.head_dim_v ? a.head_dim : a.head_dim_v;
  if (d <= 64) launch<64>(a, stream);
  else if (d <= 96) launch<96>(a, stream);
  else launch<128>(a, stream);
  return hipGetLastError();
}

}  // namespace ls
