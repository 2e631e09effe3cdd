// Internal declarations shared by the host entry points and the kernels of
// the response-replay attention library.  Not part of the public ABI.
#pragma once

// Workgroups that share K/V tiles are mapped onto one XCD (see xcd_work_item).
#ifndef LS_XCD_MAP
#define LS_XCD_MAP 1
#endif

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ls {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr int kMaxMergeGroups = 64;        // groups of one merge call (kernel arguments)
// Split bounds travel in the kernel arguments (< 4 KiB), as 32-bit offsets from
// the launch's first key (64-bit bounds took a second launch from 129 splits on).
constexpr int kMaxSplitsPerLaunch = 448;

// Most row chunks of the bf16 dk/dv kernel (partials in the backward workspace):
// up to 16 chunks of at least 128 packed rows, so that the few key blocks of a
// short response still give many workgroups, and more only where 16 would hold
// over 2,048 rows each (the partials are written and read once per chunk).
// Measured with the reduce: 77 tokens x 16 heads 59 -> 26 us, 1,111 tokens
// 140 -> 72 us.
inline int dkdv_row_chunks(int n_q, int group) {
  const int64_t rows = (int64_t)n_q * group;
  const int64_t few = (rows + 127) / 128, many = (rows + 2047) / 2048;
  return (int)(few < 16 ? few : many > 16 ? many : 16);
}
// Response keys of a workgroup of that kernel.
constexpr int kDkdvKeys = 128;
// Row chunks of a launch over n_keys keys: two workgroups per CU, or chunks of
// 2,048 rows where there are more of these.
inline int64_t dkdv_launch_chunks(int n_q, int group, int n_kv_heads, int64_t n_keys) {
  const int64_t blocks = (n_keys + kDkdvKeys - 1) / kDkdvKeys * n_kv_heads;
  const int64_t fill = (512 + blocks - 1) / blocks, many = ((int64_t)n_q * group + 2047) / 2048;
  const int64_t most = dkdv_row_chunks(n_q, group), want = fill > many ? fill : many;
  return most < want ? most : want;
}
// Most keys times chunks of any launch over up to n_resp keys: a launch of fill
// chunks has at most 512 workgroups of kDkdvKeys keys and one chunk of its keys more.
// Grows with n_q and n_resp.
inline int64_t dkdv_part_keys(int n_q, int group, int n_kv_heads, int64_t n_resp) {
  const int64_t many = ((int64_t)n_q * group + 2047) / 2048 * n_resp;
  const int64_t fill = 512 * kDkdvKeys / n_kv_heads + n_resp;
  const int64_t most = dkdv_row_chunks(n_q, group) * n_resp, want = fill > many ? fill : many;
  return most < want ? most : want;
}

// Row chunks of the fp32 matrix-core dk/dv kernel: 128 packed rows (one 32-row
// tile per wave of its workgroups), at most 16 chunks.
inline int f32_dkdv_chunks(int n_q, int group) {
  const int64_t c = ((int64_t)n_q * group + 127) / 128;
  return (int)(c < 16 ? c : 16);
}

// Packed query rows of a workgroup of the bf16 dq kernel.
constexpr int kDqRows = 128;

// Most rows (of head_dim floats) of dq partial sums that one key range's chunks
// take: 512 workgroups, two per CU, of up to 128 packed rows.  The workspace has
// room for two such ranges (dq_part_bytes).  Both grow with n_q, so that a workspace made
// for more rows serves fewer.
inline int64_t dq_part_rows(int n_q, int group) {
  const int64_t rows = (int64_t)n_q * group;
  return 512 * (rows < 128 ? rows : 128);
}
inline size_t dq_part_bytes(int n_q, int group, int head_dim) {
  return 2 * (size_t)dq_part_rows(n_q, group) * head_dim * 4;
}

// Key ranges of one dq launch: workgroups z0[i] .. z0[i + 1] - 1 (grid z) work on
// range i, chunks of `per` 32-key tiles of it.  With tail_chunks (one range, bf16)
// these are the chunks of the row tiles before tail_x; the others have tail_chunks
// chunks of tail_per tiles, and the grid is the list of both (tail last).
constexpr int kMaxDqRanges = 16;
struct DqRanges {
  int32_t n;
  int32_t tail_x = 0, tail_per = 0, tail_chunks = 0;
  int32_t z0[kMaxDqRanges + 1];
  int32_t per[kMaxDqRanges];
  int64_t begin[kMaxDqRanges], end[kMaxDqRanges];
#ifdef __HIPCC__
  __device__ __forceinline__ int of(int z) const {
    int i = 0;
    while (i + 1 < n && z >= z0[i + 1]) ++i;
    return i;
  }
#endif
};
// One range's chunks; `form` tells launches that cannot be joined apart.
struct DqPlan {
  int64_t begin, end;
  int32_t chunks, per, form;
  bool joins;               // may share a launch with other ranges (through partial sums)
  int32_t tail_x = 0, tail_per = 0, tail_chunks = 0;   // as in DqRanges
};

// Whether the fp32 matrix-core kernels take these shapes (the generic kernels
// take the others).
bool f32_mfma_fits(int head_dim, int head_dim_v, int n_kv_heads);

// Whether the generic kernels finish a small part of an fp32 backward first.  They walk
// the keys of dq and the rows of dk/dv one by one, 0.6 and 0.4 us each, where the
// matrix cores and the reduce after them take 8 and 12 us, 17 and 21 at width 128.
// Measured, generic and matrix cores, in calls of the response's keys alone: dk/dv of
// 16 rows of 64 21 and 25 us, of 24 of 16 25 and 25, of 32 of 64 29 and 26, of 48 of 128
// 46 and 44; dq of 4 keys of 64 21 and 25, of 4 of 128 30 and 42.  The generic dk/dv has
// a wave per key and KV head: 2,048 of 20 rows of 64 28 and 30 us, 4,096 32 and 30,
// 16,384 64 and 44.
inline int64_t f32_width(int head_dim, int head_dim_v) {
  const int d = head_dim > head_dim_v ? head_dim : head_dim_v;
  return d <= 64 ? 64 : d <= 96 ? 96 : 128;
}
inline bool f32_dkdv_small(int64_t width, int64_t rows, int64_t keys, int n_kv_heads) {
  return 3 * rows <= width && keys * n_kv_heads <= 2048;
}
// A dq range that shares its launch with others costs little more, and which they are
// must not change its bits: the line lies below the one for a range alone.  4 keys with
// two ranges of 1,000 and 3,096: width 64 25 us for 23, 128 35 for 29, 8 keys 40 for 32.
inline bool f32_dq_small(int64_t width, int64_t rows, int64_t keys) {
  return 32 * keys <= width || 48 * keys + 32 * rows <= 9 * width;
}

// Everything a forward-split kernel needs; passed by value as a kernel argument.
struct FwdArgs {
  const void* q;
  const void* k_pool;
  const void* v_pool;
  const int32_t* page_table;
  float* out_part;          // [n_splits, n_q, Hq, Dv]
  float* lse_part;          // [n_splits, Hq, n_q]
  int64_t q_pos0;
  int64_t k_pos_stride;     // elements between positions in a K page (Hkv * D)
  int64_t v_pos_stride;     // elements between positions in a V page (Hkv * Dv)
  int32_t n_q, n_q_heads, n_kv_heads, group, log2_group;
  int32_t head_dim, head_dim_v;
  int32_t log2_page;
  float scale_log2;         // softmax_scale * log2(e)
  int32_t n_splits;
  int64_t split_base, split_more;   // split_more: added to every end (a split past 32 bits)
  uint32_t split_lo[kMaxSplitsPerLaunch], split_hi[kMaxSplitsPerLaunch];
  __host__ __device__ int64_t split_begin(int i) const { return split_base + split_lo[i]; }
  __host__ __device__ int64_t split_end(int i) const { return split_base + split_hi[i] + split_more; }
};
static_assert(sizeof(FwdArgs) <= 4096, "kernel arguments");

// Puts the first of n sorted splits (with kv_begin and kv_end) into a's arguments: as
// many as these hold and 32-bit offsets reach, or one longer split alone.  Returns
// how many.
template <typename Split>
inline int pack_splits(FwdArgs& a, const Split* splits, int n) {
  a.split_base = splits[0].kv_begin;
  a.split_more = 0;
  a.n_splits = 0;
  while (a.n_splits < kMaxSplitsPerLaunch && a.n_splits < n &&
         splits[a.n_splits].kv_end - a.split_base <= (int64_t)UINT32_MAX) {
    a.split_lo[a.n_splits] = (uint32_t)(splits[a.n_splits].kv_begin - a.split_base);
    a.split_hi[a.n_splits] = (uint32_t)(splits[a.n_splits].kv_end - a.split_base);
    ++a.n_splits;
  }
  if (a.n_splits == 0) {
    a.split_lo[0] = a.split_hi[0] = 0;
    a.split_more = splits[0].kv_end - a.split_base;
    a.n_splits = 1;
  }
  return a.n_splits;
}

// An estimate of a forward launch's time in workgroups of rows_per packed rows, one
// per CU each, that take `tile` for 32 keys and `ends` to start and end: the rounds of
// 256 workgroups that the long splits take (those of half the longest one's time or
// more), or all workgroups' time shared among the CUs where that is more.
inline double fwd_time(const FwdArgs& a, int rows_per, double tile, double ends) {
  const int64_t wgs = ((int64_t)a.n_q * a.group + rows_per - 1) / rows_per * a.n_kv_heads;
  auto one = [&](int i) { return tile * (double)((a.split_end(i) - a.split_begin(i) + 31) / 32) + ends; };
  double most = 0, sum = 0;
  for (int i = 0; i < a.n_splits; ++i) most = one(i) > most ? one(i) : most;
  int64_t longs = 0;
  for (int i = 0; i < a.n_splits; ++i) {
    longs += 2 * one(i) >= most;
    sum += one(i);
  }
  const double rounds = (double)((longs * wgs + 255) / 256) * most, shared = sum * (double)wgs / 256;
  return rounds > shared ? rounds : shared;
}

// Whether the fp32 matrix-core forward takes 128-row workgroups, or 32-row ones whose
// four waves share the keys.  A tile and the ends (start, merge of the waves) take 4.5
// and 4 us with 128 rows, 1.77 and 5 with 32, at width 128 (at 64 0.55 of that).
// Measured at width 128, workgroups of 128 and of 32 rows: 6 and 24 with 256 keys each
// 44 and 21 us; 120 and 460 46 and 43, with 64 keys 18 and 27, with 4,096 keys 622 and
// 467; 216 and 828 48 and 81, 20 and 51, 627 and 912; 288 and 1,104 81 and 100, 31 and
// 64, 1,125 and 1,141 (168 points: within 3% of the better one in all but 3, at most
// 6% off; 32 rows wherever 128-row workgroups were fewer than the CUs: in all but 52,
// up to 2.7 times).
inline bool f32_fwd_wide(const FwdArgs& a) { return fwd_time(a, 128, 4.5, 4) < fwd_time(a, 32, 1.77, 5); }

// Backward.  The dq launches take their key ranges from DqRanges, the dk/dv ones
// from kv_begin / kv_end.
struct BwdArgs {
  const void* q;
  const void* k_pool;
  const void* v_pool;
  const int32_t* page_table;
  const void* d_out;
  const float* delta;       // [Hq, n_q]  d_out . out
  const float* lse2;        // [Hq, n_q]  lse * log2(e); +inf for rows with no key
  float* dq;                // [n_q, Hq, D]
  float* dk_resp;           // [kv_len - prefix_len, Hkv, D]
  float* dv_resp;           // [kv_len - prefix_len, Hkv, Dv]
  float* dkdv_part;         // partial dk/dv sums of row chunks over the launch's keys (bf16:
                            // [row chunks, 2, Hkv, keys, D]; fp32: [row chunks, keys, Hkv, D + Dv])
  float* dq_part;           // partial dq sums of key chunks [chunks, n_q, Hq, D], unscaled
                            // (dq_part_bytes in all)
  int64_t q_pos0;
  int64_t prefix_len;
  int64_t kv_begin, kv_end;
  int64_t k_pos_stride, v_pos_stride;
  int32_t n_q, n_q_heads, n_kv_heads, group, log2_group;
  int32_t head_dim, head_dim_v;
  int32_t log2_page;
  float scale;              // softmax_scale
  float scale_log2;         // softmax_scale * log2(e)
  int32_t accumulate_dq, accumulate_dkv;
  int32_t dkdv_rows;        // bf16 path: packed rows per dk/dv chunk, a multiple of 32 (set by
                            // the launcher)
};

// DSA index scores (Eq. dsa-index) over positions [pos_begin, pos_end).
struct DsaArgs {
  const void* q;             // [n_q, n_heads, 128] bf16 index queries
  const float* w;            // [n_q, n_heads] head weights
  const void* k_pool;        // [n_phys, page, 128] bf16 index keys, one per position
  const int32_t* page_table;
  float* scores;             // [n_q, ld]: I[t, s] at t * ld + (s - pos_begin)
  int64_t ld, pos_begin, pos_end;
  int64_t chunk;             // positions per workgroup, a multiple of 32 (set by the launcher)
  int32_t n_q, n_heads, log2_page;
};

// Top-k of each row of a score matrix (Eq. glm-global-dsa).
struct TopkArgs {
  const float* scores;       // [n_rows, ld]
  const int32_t* positions;  // [n_rows, ld] or null (position = pos_offset + column)
  int32_t* out_pos;          // [n_rows, out_ld], k used per row
  float* out_scores;         // [n_rows, out_ld] or null
  int64_t ld, out_ld, n, pos_offset;
  int64_t seg;               // columns per workgroup (set by the launcher)
  int32_t n_rows, k;
};

// Sparse latent replay (one shared latent row per position, 576 / 512 wide).
struct SparseArgs {
  const void* q;             // [n_q, H, 576] bf16
  const void* latent;        // pool [n_phys, S, 1, 576] bf16
  const int32_t* page_table;
  const int32_t* idx;        // [n_q, topk] selected prefix positions (others: no key)
  int32_t* phys;             // workspace [n_q, n_max] physical latent rows
  int32_t* ntok;             // workspace [n_q] keys in each token's list
  float* out;                // [n_q, H, 512] fp32 normalized
  float* lse;                // [H, n_q]
  const void* d_out;         // [n_q, H, 512] bf16
  const float* delta;        // [H, n_q]
  const float* lse2;         // [H, n_q]
  float* dq;                 // [n_q, H, 576]
  int64_t prefix_len, kv_len, window0;   // window0 = q_pos0 - prefix_len
  int32_t n_q, n_heads, topk, n_max, log2_page;
  float scale, scale_log2;
  int32_t accumulate_dq;
};

// Launchers (return the hipError_t of the launch).
hipError_t launch_sparse_phys(const SparseArgs& a, hipStream_t stream);
// n_chunks > 1: a.out / a.lse ([chunks, ...]) or a.dq ([chunks, n_q, H, 576]) hold
// the partial results of each token's key chunks
hipError_t launch_sparse_fwd(const SparseArgs& a, int n_chunks, hipStream_t stream);
hipError_t launch_sparse_bwd(const SparseArgs& a, int n_chunks, hipStream_t stream);
hipError_t launch_gather(const void* k_pool, const void* v_pool, const int32_t* page_table,
                         int64_t pos_begin, int64_t pos_end, int log2_page, int64_t k_row_elems,
                         int64_t v_row_elems, int esize, void* k_out, void* v_out,
                         hipStream_t stream);
hipError_t launch_scatter(void* k_pool, void* v_pool, const int32_t* page_table,
                          int64_t pos_begin, int64_t pos_end, int log2_page, int64_t k_row_elems,
                          int64_t v_row_elems, int esize, const void* k_src, const void* v_src,
                          hipStream_t stream);
// Parts begin[k] .. end[k] - 1 (host arrays, non-empty) compose group k; with
// several groups their results go to group_out / group_lse and the groups
// compose out / lse, in order.
hipError_t launch_merge(const float* out_part, const float* lse_part, const int32_t* begin,
                        const int32_t* end, int n_groups, int n_q, int n_heads, int dv,
                        bool out_bf16, bool bf16_numerator, float* group_out, float* group_lse,
                        void* out, float* lse, hipStream_t stream);
hipError_t launch_fwd_f32(const FwdArgs& a, hipStream_t stream);
// fp32 on the matrix cores, for the shapes f32_mfma_fits accepts (launch_fwd_f32 and
// the backward entry point take them for those, the generic kernels for the others)
hipError_t launch_fwd_f32_mfma(const FwdArgs& a, hipStream_t stream);
DqPlan plan_dq_f32_mfma(const BwdArgs& a, int64_t begin, int64_t end);
hipError_t launch_dq_f32_mfma(const BwdArgs& a, const DqRanges& r, int form, float* part,
                              hipStream_t stream);
// dk/dv of the keys from key0 to a.kv_end
hipError_t launch_dkdv_f32_mfma(const BwdArgs& a, int64_t key0, hipStream_t stream);
// dq (+)= scale * the sum of each range's partials (n values each, a multiple of 4), in order
hipError_t launch_dq_reduce(const float* part, const DqRanges& r, int64_t n, float scale,
                            bool accumulate, float* dq, hipStream_t stream);
hipError_t launch_hbm_read(const void* buf, int64_t n16, uint32_t* out, hipStream_t stream);
hipError_t launch_dsa_scores(const DsaArgs& a, hipStream_t stream);
// n_chunks > 1 (from topk_chunks): the rows' chunks are selected from first, into
// cand_pos / cand_scores [n_rows, n_chunks * k]
int topk_chunks(int64_t n_rows, int64_t n, int k);
hipError_t launch_topk(const TopkArgs& a, int n_chunks, int32_t* cand_pos, float* cand_scores,
                       hipStream_t stream);
hipError_t launch_fwd_bf16_d256(const FwdArgs& a, hipStream_t stream);
hipError_t launch_bwd_prep(const void* d_out, const void* out, bool dout_bf16, bool out_bf16,
                           const float* lse, int n_q, int n_heads, int dv, float* delta,
                           float* lse2, hipStream_t stream);
// the generic fp32 kernels: dq over [a.kv_begin, a.kv_end), dk/dv of its keys from key0 on
hipError_t launch_dq_f32_generic(const BwdArgs& a, hipStream_t stream);
hipError_t launch_dkdv_f32_generic(const BwdArgs& a, int64_t key0, hipStream_t stream);
DqPlan plan_dq_bf16_d256(const BwdArgs& a, int64_t begin, int64_t end);
hipError_t launch_dq_bf16_d256(const BwdArgs& a, const DqRanges& r, float* part,
                               hipStream_t stream);
hipError_t launch_dkdv_bf16_d256(const BwdArgs& a, int64_t key0, hipStream_t stream);

}  // namespace ls
