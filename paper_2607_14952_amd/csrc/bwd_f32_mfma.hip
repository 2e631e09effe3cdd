// fp32 backward on the matrix cores (f32_mfma.h) for head dimensions that are
// multiples of 4 up to 128, any GQA group: products and sums in fp32 as the
// generic kernels form them.
//
// dq.  A workgroup is 4 waves = kRW groups of 32 packed query rows of one KV
// head x 4 / kRW key slots, over one chunk of the key range.  Per iteration it
// stages 4 / kRW 32-key tiles of K and V in LDS; each wave forms, for its rows
// and its slot's tile,
//   S^T = K Q^T, dP^T = V dO^T, P = exp2(S * scale * log2(e) - lse2),
//   dS = P (dP - Delta), dq^T += K^T dS^T.
// Key slots are added through LDS, chunks by a reduce kernel, both in order
// (deterministic).
//
// dk/dv.  A workgroup owns 32 response keys of one KV head (lane j: key j; its
// K and V rows stay in registers) and one chunk of the packed query rows; each
// of its 4 waves takes every fourth 32-row tile of the chunk:
//   S = Q K^T, dP = dO V^T, dv^T += dO^T P, dk^T += Q^T dS.
// The waves are added through LDS, the chunks by a reduce kernel, in order.
//
// Both are bound by the MFMAs (64 cycles each) once every SIMD has a wave, which
// the chunk counts below see to.  Measured against the scalar kernels: 128 rows
// x 4,096 keys, 2 heads of 64, dq + dk/dv 2,900 -> 38 us; 500 rows x 16,001
// keys, 8 heads of 128 on 2 KV heads 25.8 -> 0.55 ms (dq at 100 TFLOP/s of the
// 154 an fp32 GEMM reaches: the matrix cores are busy 73% of the time, with two
// waves per SIMD where four row groups share a tile; with one, 0.61 ms).
#include <math.h>

#include <algorithm>

#include "f32_mfma.h"

namespace ls {
namespace {
using namespace f32m;

// ============================================================== dq
template <int kDP, int kRW>
__global__ __launch_bounds__(256, kRW == 4 ? 2 : 1) void bwd_dq_f32_mfma_kernel(
    BwdArgs a, DqRanges ranges, float* __restrict__ part) {
  constexpr int kKW = 4 / kRW;
  constexpr int kS = kRowS<kDP>;
  constexpr int kDB = kDP / 32;
  __shared__ __attribute__((aligned(16))) float smem[2 * kKW * 32 * kS];
  float* const ks = smem;
  float* const vs = smem + kKW * 32 * kS;

  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int rw = w % kRW, kw = w / kRW;
  const int j = lane & 31, h = lane >> 5;
  const int g = blockIdx.y, z = blockIdx.z;   // z: a chunk of one of the key ranges
  const int G = a.group, D = a.head_dim, Dv = a.head_dim_v;
  const int64_t rows_total = (int64_t)a.n_q * G;
  const int64_t row0 = (int64_t)blockIdx.x * (32 * kRW);
  const int64_t prow = row0 + rw * 32 + j;
  const bool row_ok = prow < rows_total;
  const int tok = (int)(prow / G);
  const int head = g * G + (int)(prow - (int64_t)tok * G);
  const int tok_last = (int)(min(rows_total, row0 + 32 * kRW) - 1) / G;
  const int ri = ranges.of(z);
  const int64_t kb = ranges.begin[ri], kv_end = ranges.end[ri];
  const int64_t k_hi = min(kv_end, a.q_pos0 + tok_last + 1);
  const int64_t my_lim = row_ok ? min(kv_end, a.q_pos0 + tok + 1) : kb;
  // below: visible to every row (of a whole row group)
  const int64_t k_all =
      row0 + 32 * kRW <= rows_total ? min(kv_end, a.q_pos0 + (int)(row0 / G) + 1) : kb;
  const int64_t k_lo = kb & ~int64_t(31);
  const int all_tiles = k_hi > kb ? (int)((k_hi - k_lo + 31) / 32) : 0;
  const int t_begin = min(all_tiles, (z - ranges.z0[ri]) * ranges.per[ri]);
  const int t_end = min(all_tiles, t_begin + ranges.per[ri]);

  const int64_t rh = row_ok ? (int64_t)tok * a.n_q_heads + head : 0;   // (rows past the end: row 0)
  float qv[kDP / 2], dov[kDP / 2];
  load_half_row<kDP>(qv, static_cast<const float*>(a.q) + rh * D, D, h);
  load_half_row<kDP>(dov, static_cast<const float*>(a.d_out) + rh * Dv, Dv, h);
  const int64_t stat = row_ok ? (int64_t)head * a.n_q + tok : 0;
  const float lse2 = a.lse2[stat], delta = a.delta[stat];
  f32x16 acc[kDB];
#pragma unroll
  for (int b = 0; b < kDB; ++b) acc[b] = zero16();

  // (128-wide rows with two waves per SIMD leave no registers to load ahead)
  constexpr bool kPre = !(kDP == 128 && kRW == 4);
  KvStage<kDP, kKW> stage;
  if (kPre && t_begin < t_end) {
    stage.load_pages(a, k_lo + (int64_t)t_begin * 32, kb, k_hi, tid);
    stage.load(a, g, k_lo + (int64_t)t_begin * 32, kb, k_hi, tid);
  }
  for (int t = t_begin; t < t_end; t += kKW) {
    const int64_t t0 = k_lo + (int64_t)t * 32;
    if (!kPre) {
      stage.load_pages(a, t0, kb, k_hi, tid);
      stage.load(a, g, t0, kb, k_hi, tid);
    }
    __syncthreads();   // every wave is done with the previous tiles
    stage.template store<kS, kS>(a, ks, vs, tid);
    __syncthreads();
    if (kPre && t + kKW < t_end) stage.load(a, g, t0 + 32 * kKW, kb, k_hi, tid);
    if (t + kw >= t_end) continue;   // (uniform per wave; the barriers above are not skipped)

    const int64_t tw = t0 + 32 * kw;
    f32x16 s, dp;
    row_products<kDP, kS>(ks + kw * 32 * kS, qv, s, vs + kw * 32 * kS, dov, dp, j, h);
#pragma unroll
    for (int r = 0; r < 16; ++r)
      s[r] = __builtin_amdgcn_exp2f(fmaf(s[r], a.scale_log2, -lse2)) * (dp[r] - delta);
    if (tw < kb || tw + 32 > k_all) {
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (!in_rows(r, h, kb - tw, my_lim - tw)) s[r] = 0.f;
    }
    col_product<kDP, kS>(ks + kw * 32 * kS, s, acc, j, h);
  }

  if constexpr (kKW > 1) {
    constexpr int kAcc = kDB * 16 * 64;
    static_assert((kKW - 1) * kAcc <= 2 * kKW * 32 * kS, "slot sums");
    __syncthreads();
    if (kw > 0) acc_to_lds<kDB>(smem + (kw - 1) * kAcc, acc, lane);
    __syncthreads();
    if (kw > 0) return;
#pragma unroll
    for (int k = 1; k < kKW; ++k) acc_add_lds<kDB>(acc, smem + (k - 1) * kAcc, 1.f, lane);
  }
  // a chunk's partial sum (unscaled), or the result when there is one chunk
  float* const out = part ? part + (int64_t)z * a.n_q * a.n_q_heads * D : a.dq;
  const float c = part ? 1.f : a.scale;
  const bool add = !part && a.accumulate_dq;
  // rows to form again key by key (f32_rows.h); the rows past the end are none
  uint32_t again = not_finite<kDB>(acc) & (uint32_t)__ballot(row_ok);
  if (row_ok && !(add && (again >> j & 1))) {
    float* dst = out + rh * D;
#pragma unroll
    for (int b = 0; b < kDB; ++b) {
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const int d = 32 * b + 8 * q4 + 4 * h;
        f32x4 v = {0.f, 0.f, 0.f, 0.f};
        if (add) v = load_piece(dst, d, D);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = fmaf(c, acc[b][4 * q4 + e], v[e]);
        if (d < D) *reinterpret_cast<f32x4*>(dst + d) = v;
      }
    }
  }
  if (__builtin_expect(again != 0, 0)) {
    __threadfence();   // (the values stored so far come first)
    for (; again; again &= again - 1) {
      const int64_t r = of_lane(rh, __builtin_ctz(again));
      const int t = (int)(r / a.n_q_heads), hd = (int)(r - (int64_t)t * a.n_q_heads);
      const int zz = opaque(blockIdx.z), i = ranges.of(zz), ln = lane_id();
      const int64_t begin = ranges.begin[i];
      const int64_t from = (begin & ~int64_t(31)) + (int64_t)(zz - ranges.z0[i]) * ranges.per[i] * 32;
      float x[2];
      f32r::dq_row<2>(a, max(begin, from),
                      min(min(ranges.end[i], a.q_pos0 + t + 1), from + ranges.per[i] * 32), t, hd,
                      ln, x);
      float* dst = out + r * D;
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const int d = ln + 64 * k;
        if (d < D) dst[d] = fmaf(c, x[k], add ? dst[d] : 0.f);
      }
    }
  }
}

// ============================================================== dk/dv
// First packed row (a multiple of 32) of the chunk that sees a key of the
// 32-key block at j0, and the chunk's end; active when lo < hi.
__device__ __forceinline__ void chunk_rows(const BwdArgs& a, int64_t j0, int chunk, int rows_per,
                                           int64_t& lo, int64_t& hi) {
  const int64_t rows_total = (int64_t)a.n_q * a.group;
  const int64_t first_tok = j0 > a.q_pos0 ? j0 - a.q_pos0 : 0;
  const int64_t vis = min(rows_total, first_tok * a.group) & ~int64_t(31);
  lo = max((int64_t)chunk * rows_per, vis);
  hi = min(rows_total, (int64_t)(chunk + 1) * rows_per);
}

template <int kDP>
__global__ __launch_bounds__(256) void bwd_dkdv_f32_mfma_kernel(BwdArgs a, int64_t key0,
                                                                int rows_per,
                                                                float* __restrict__ part) {
  constexpr int kS = kRowS<kDP>;
  constexpr int kDB = kDP / 32;
  __shared__ __attribute__((aligned(16))) float smem[4 * 2 * 32 * kS + 4 * 64];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int j = lane & 31, h = lane >> 5;
  const int g = blockIdx.y, chunk = blockIdx.z;
  const int G = a.group, D = a.head_dim, Dv = a.head_dim_v;
  const int64_t rows_total = (int64_t)a.n_q * G;
  const int64_t j0 = key0 + (int64_t)blockIdx.x * 32;
  const int64_t key = j0 + j;
  const bool key_ok = key < a.kv_end;
  int64_t row_lo, row_hi;
  chunk_rows(a, j0, chunk, rows_per, row_lo, row_hi);
  if (row_lo >= row_hi) return;

  float kv[kDP / 2], vv[kDP / 2];
  {
    // (keys past the end: the last one; nothing is stored for them)
    const int64_t pr = phys_pos(a.page_table, min(key, a.kv_end - 1), a.log2_page);
    load_half_row<kDP>(kv, static_cast<const float*>(a.k_pool) + pr * a.k_pos_stride + (int64_t)g * D,
                       D, h);
    load_half_row<kDP>(vv, static_cast<const float*>(a.v_pool) + pr * a.v_pos_stride + (int64_t)g * Dv,
                       Dv, h);
  }
  f32x16 dk[kDB], dv[kDB];
#pragma unroll
  for (int b = 0; b < kDB; ++b) dk[b] = dv[b] = zero16();

  // Each wave stages and reads its own tiles (no barrier): rows past the chunk's
  // end repeat its last one and get P = 0.
  float* const qs = smem + w * 2 * 32 * kS;
  float* const ds = qs + 32 * kS;
  float* const st = smem + 4 * 2 * 32 * kS + 64 * w;   // 32 lse2, 32 Delta
  for (int64_t rt = row_lo + 32 * w; rt < row_hi; rt += 128) {
    constexpr int kPieces = kDP / 8;
    f32x4 q[kPieces], d[kPieces];
#pragma unroll
    for (int i = 0; i < kPieces; ++i) {
      const int idx = lane + 64 * i;
      const int row = idx / (kDP / 4), c = 4 * (idx % (kDP / 4));
      const int64_t prow = min(rt + row, row_hi - 1);
      const int tok = (int)(prow / G);
      const int64_t rh = (int64_t)tok * a.n_q_heads + g * G + (prow - (int64_t)tok * G);
      q[i] = load_piece(static_cast<const float*>(a.q) + rh * D, c, D);
      d[i] = load_piece(static_cast<const float*>(a.d_out) + rh * Dv, c, Dv);
    }
    float x;
    {
      const int64_t prow = min(rt + j, row_hi - 1);
      const int tok = (int)(prow / G);
      const int64_t o = (g * G + (prow - (int64_t)tok * G)) * a.n_q + tok;
      x = (h ? a.delta : a.lse2)[o];
      if (!h && rt + j >= row_hi) x = INFINITY;
    }
#pragma unroll
    for (int i = 0; i < kPieces; ++i) {
      const int idx = lane + 64 * i;
      const int row = idx / (kDP / 4), c = 4 * (idx % (kDP / 4));
      *reinterpret_cast<f32x4*>(qs + row * kS + c) = pad(q[i], c, D);
      *reinterpret_cast<f32x4*>(ds + row * kS + c) = pad(d[i], c, Dv);
    }
    st[lane] = x;

    f32x16 p, dp;
    row_products<kDP, kS>(qs, kv, p, ds, vv, dp, j, h);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int row = row_of(r, h);
      const int64_t tok = (rt + row) / G;
      const float e = __builtin_amdgcn_exp2f(fmaf(p[r], a.scale_log2, -st[row]));
      p[r] = a.q_pos0 + tok >= key ? e : 0.f;
      dp[r] = p[r] * (dp[r] - st[32 + row]);
    }
    col_product<kDP, kS>(ds, p, dv, j, h);
    col_product<kDP, kS>(qs, dp, dk, j, h);
  }

  constexpr int kAcc = kDB * 16 * 64;
  static_assert(3 * 2 * kAcc <= 4 * 2 * 32 * kS, "wave sums");
  __syncthreads();
  if (w > 0) {
    acc_to_lds<kDB>(smem + (2 * (w - 1)) * kAcc, dk, lane);
    acc_to_lds<kDB>(smem + (2 * (w - 1) + 1) * kAcc, dv, lane);
  }
  __syncthreads();
  if (w > 0) return;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    acc_add_lds<kDB>(dk, smem + 2 * k * kAcc, 1.f, lane);
    acc_add_lds<kDB>(dv, smem + (2 * k + 1) * kAcc, 1.f, lane);
  }
  // part[chunk][key - key0][g][D + Dv]
  auto part_of = [&](int64_t k) {
    return part + (((int64_t)chunk * (a.kv_end - key0) + (k - key0)) * a.n_kv_heads + g) * (D + Dv);
  };
  if (key_ok) {
    float* dst = part_of(key);
#pragma unroll
    for (int b = 0; b < kDB; ++b) {
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const int d = 32 * b + 8 * q4 + 4 * h;
        f32x4 x, y;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          x[e] = dk[b][4 * q4 + e];
          y[e] = dv[b][4 * q4 + e];
        }
        if (d < D) *reinterpret_cast<f32x4*>(dst + d) = x;
        if (d < Dv) *reinterpret_cast<f32x4*>(dst + D + d) = y;
      }
    }
  }
  // keys to form again row by row (f32_rows.h); the keys past the end are none
  uint32_t again = (not_finite<kDB>(dk) | not_finite<kDB>(dv)) & (uint32_t)__ballot(key_ok);
  if (__builtin_expect(again != 0, 0)) {
    __threadfence();   // (the values stored so far come first)
    for (; again; again &= again - 1) {
      const int64_t k = of_lane(key, __builtin_ctz(again));
      const int ln = lane_id();
      float x[2], y[2];
      f32r::dkdv_key<2>(a, k, g, row_lo, row_hi, ln, x, y);
      float* dst = part_of(k);
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int d = ln + 64 * i;
        if (d < D) dst[d] = x[i];
        if (d < Dv) dst[D + d] = y[i];
      }
    }
  }
}

// Adds the chunks of a key's dk and dv in order; thread = 4 channels of one
// (key, KV head).
__global__ __launch_bounds__(256) void dkdv_f32_reduce_kernel(BwdArgs a, int64_t key0,
                                                              int n_chunks, int rows_per,
                                                              const float* __restrict__ part) {
  const int D = a.head_dim, W = D + a.head_dim_v;
  const int64_t n_keys = a.kv_end - key0;
  const int64_t item = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (item >= n_keys * a.n_kv_heads * (W / 4)) return;
  const int64_t kg = item / (W / 4);                 // (key, g)
  const int c = (int)(item - kg * (W / 4)) * 4;
  const int64_t jj = kg / a.n_kv_heads;
  const int64_t j0 = key0 + (jj & ~int64_t(31));
  f32x4 sum = {0.f, 0.f, 0.f, 0.f};
  for (int k = 0; k < n_chunks; ++k) {
    int64_t lo, hi;
    chunk_rows(a, j0, k, rows_per, lo, hi);
    if (lo < hi)
      sum += *reinterpret_cast<const f32x4*>(part + ((int64_t)k * n_keys * a.n_kv_heads + kg) * W + c);
  }
  const int64_t row = (key0 - a.prefix_len) * a.n_kv_heads + kg;
  float* dst = c < D ? a.dk_resp + row * D + c : a.dv_resp + row * a.head_dim_v + (c - D);
  if (c < D) sum *= a.scale;
  if (a.accumulate_dkv) sum += *reinterpret_cast<const f32x4*>(dst);
  *reinterpret_cast<f32x4*>(dst) = sum;
}

template <int kDP>
void launch_dq(const BwdArgs& a, const DqRanges& r, bool share, float* part, hipStream_t stream) {
  const int64_t rows = (int64_t)a.n_q * a.group;
  if (share)
    hipLaunchKernelGGL((bwd_dq_f32_mfma_kernel<kDP, 4>),
                       dim3((unsigned)((rows + 127) / 128), a.n_kv_heads, r.z0[r.n]), dim3(256), 0,
                       stream, a, r, part);
  else
    hipLaunchKernelGGL((bwd_dq_f32_mfma_kernel<kDP, 1>),
                       dim3((unsigned)((rows + 31) / 32), a.n_kv_heads, r.z0[r.n]), dim3(256), 0,
                       stream, a, r, part);
}

template <int kDP>
hipError_t launch_dkdv(const BwdArgs& a, int64_t key0, hipStream_t stream) {
  const int n_chunks = f32_dkdv_chunks(a.n_q, a.group);
  const int64_t rows = (int64_t)a.n_q * a.group;
  const int rows_per = (int)((rows + n_chunks - 1) / n_chunks + 31) / 32 * 32;
  const int64_t n_keys = a.kv_end - key0;
  hipLaunchKernelGGL(bwd_dkdv_f32_mfma_kernel<kDP>,
                     dim3((unsigned)((n_keys + 31) / 32), a.n_kv_heads, n_chunks), dim3(256), 0,
                     stream, a, key0, rows_per, a.dkdv_part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int64_t items = n_keys * a.n_kv_heads * ((a.head_dim + a.head_dim_v) / 4);
  hipLaunchKernelGGL(dkdv_f32_reduce_kernel, dim3((unsigned)((items + 255) / 256)), dim3(256), 0,
                     stream, a, key0, n_chunks, rows_per, a.dkdv_part);
  return hipGetLastError();
}

}  // namespace

DqPlan plan_dq_f32_mfma(const BwdArgs& a, int64_t begin, int64_t end) {
  const int64_t rows = (int64_t)a.n_q * a.group;
  const int64_t n_tiles = (end - (begin & ~int64_t(31)) + 31) / 32;
  const int64_t wide = (rows + 127) / 128 * a.n_kv_heads, narrow = (rows + 31) / 32 * a.n_kv_heads;
  // Chunks of at least 8 (4) key tiles, enough for two workgroups on each CU
  // and no more than the partial sums have room for.  Four row groups share
  // a staged tile where that still gives nearly every CU its two workgroups: 32-row
  // ones in more rounds are slower where the sums have room for 456 (600 tokens x 24
  // heads on 3 over 30,000 keys: 4,390 us, shared 3,215) or 510 (516 x 8 on 2 over
  // 16,001: 912 and 573; 260 x 24 on 3 over 30,000: 1,665 and 971).
  const int64_t room = std::max<int64_t>(1, dq_part_rows(a.n_q, a.group) / ((int64_t)a.n_q * a.n_q_heads));
  const int64_t most = std::min(room, (n_tiles + 7) / 8);
  const bool share = wide * most >= 448;
  int64_t want = 1;
  if (share) {
    // Of the counts that fill one to three rounds of two workgroups per CU, the
    // least tiles a CU takes one after another (a last round of single workgroups
    // takes 0.6 of the time; 3 tiles for a start and end).  One workgroup more than
    // a round holds costs a round: 200 tokens x 16 heads on 2 over 20,000 keys, 520
    // workgroups 304 us, 494 261; 600 x 3 on 3 over 10,000 135 and 119.
    double least = INFINITY;
    for (int64_t k = 0; k <= 3; ++k) {
      const int64_t c = std::max<int64_t>(1, std::min(512 * k / wide, most));
      const int64_t n = wide * c, last = n % 512;
      const double cost = ((double)(n / 512) + (last == 0 ? 0. : last <= 256 ? 0.6 : 1.)) *
                          ((double)((n_tiles + c - 1) / c) + 3);
      if (cost < least) {
        least = cost;
        want = c;
      }
    }
  } else {
    want = std::max<int64_t>(1, std::min({(512 + narrow - 1) / narrow, (n_tiles + 3) / 4, room}));
  }
  const int64_t items = share ? wide : narrow;
  const int64_t unit = share ? 1 : 4;                // whole iterations of the workgroup
  const int64_t per = ((n_tiles + want - 1) / want + unit - 1) / unit * unit;
  const int64_t chunks = (n_tiles + per - 1) / per;
  // (128 rows, 3 ranges: 63 us apart, 49 in one launch; 500 rows, 590 and 586)
  return DqPlan{begin, end, (int32_t)chunks, (int32_t)per, share ? 1 : 0,
                chunks > 1 || items < 128};
}

hipError_t launch_dq_f32_mfma(const BwdArgs& a, const DqRanges& r, int form, float* part,
                              hipStream_t stream) {
  const int d = a.head_dim > a.head_dim_v ? a.head_dim : a.head_dim_v;
  if (d <= 64) launch_dq<64>(a, r, form == 1, part, stream);
  else if (d <= 96) launch_dq<96>(a, r, form == 1, part, stream);
  else launch_dq<128>(a, r, form == 1, part, stream);
  return hipGetLastError();
}

hipError_t launch_dkdv_f32_mfma(const BwdArgs& a, int64_t key0, hipStream_t stream) {
  const int d = a.head_dim > a.head_dim_v ? a.head_dim : a.head_dim_v;
  return d <= 64   ? launch_dkdv<64>(a, key0, stream)
         : d <= 96 ? launch_dkdv<96>(a, key0, stream)
                   : launch_dkdv<128>(a, key0, stream);
}

}  // namespace ls
