// bf16 backward for head_dim = 256 on gfx950 (prefix held as stop-gradient
// state, Eq. gradient-boundary; dq composed over key ranges, Eq. qwen-dq-reduce).
//
// dq kernel: workgroup = 4 waves = 128 packed query rows of one KV head, lane
// l owns row l % 32.  Per 32-key tile it recomputes S^T = K Q^T, forms
// P = exp2(s*scale*log2e - lse2) with the merged log-normalizer, dP^T = V dO^T,
// dS = P (dP - Delta) and accumulates dq^T += K^T dS^T.  K and V tiles arrive
// by direct global->LDS loads into a four-slot ring, two tiles ahead
// (row-major, swizzled);
// the K^T operand of the third product comes from transposing LDS reads of
// the same K tile.  The dq product of tile t-1 is issued in the same block as
// the exponentials of tile t; its last two MFMAs run after the next tile
// barrier (every LDS read of a step lands before its barrier, since the stage
// issued after it may refill the slot).
//
// dk/dv kernel: 128 response keys of one KV head per workgroup (lane l of
// wave w owns key 32w + l % 32) against one chunk of packed query rows; Q and
// dO row tiles stream through LDS and are read row-wise for S = Q K^T and
// dP = dO V^T and transposed for dv^T += dO^T P and dk^T += Q^T dS.  Chunk
// partials are summed by a reduce kernel.  Only keys >= prefix_len ever get a
// gradient.
#include <math.h>

#include <algorithm>

#include "ls_internal.h"
#include "mfma_common.h"

namespace ls {
namespace {

constexpr int kD = 256;

// ============================================================== dq kernel
constexpr int kQBM = kDqRows;
constexpr int kQBN = kTileKeys;                   // 32
constexpr int kRowBytes = kD * 2;                 // 512 B: one key row
constexpr int kQStage = 2 * kTileBytes;           // K tile + V tile (row-major, swizzled)
#ifndef LS_DQ_AHEAD
#define LS_DQ_AHEAD 2
#endif
constexpr int kQAhead = LS_DQ_AHEAD;              // tiles in flight beyond the one consumed
constexpr int kQSlots = kQAhead + 2;

// Operand reads run a fixed number of MFMAs ahead of their use (see mfma_fence).
constexpr int kSDAhead = 2;   // steps of (K row, V row) reads in flight
#ifndef LS_DQ_KTAHEAD
#define LS_DQ_KTAHEAD 3
#endif
constexpr int kKTAhead = LS_DQ_KTAHEAD;   // transposed K operands in flight (two reads each)

#ifndef LS_DQ_KT_EARLY
#define LS_DQ_KT_EARLY 1
#endif
// Every step waits for its LDS reads before its barrier: the stage issued
// right after a barrier may refill the slot whose transposed K the step before
// it read.  The last kDqDefer MFMAs of a tile's dq product then run at the
// start of the next step, right after its first K/V operand reads are issued,
// so that the matrix core covers those reads' latency; they carry their K^T
// operands and the tile's dS across the barrier.
#ifndef LS_DQ_DEFER
#define LS_DQ_DEFER 2
#endif
constexpr int kDqDefer = LS_DQ_DEFER;
// (the shortened product loop still reads every operand only if the deferred
// MFMAs are no more than its read-ahead)
static_assert(kDqDefer >= 0 && kDqDefer <= kKTAhead, "deferred dq MFMAs");
struct DqTail {
  bf16x8 kt[kDqDefer > 0 ? kDqDefer : 1];
  bf16x8 d0, d1;
  // dq^T += the deferred products (operand 16 - kDqDefer + j)
  __device__ __forceinline__ void run(f32x16* acc) const {
#pragma unroll
    for (int j = 0; j < kDqDefer; ++j) {
      const int i = 16 - kDqDefer + j;
      acc[i >> 1] = mfma32(kt[j], (i & 1) ? d1 : d0, acc[i >> 1]);
    }
  }
};

// S^T = K Q^T and dP^T = V dO^T for one 32-key tile.  After step ks < 8,
// load(ks) issues one instruction of the next stage's direct loads; after the
// last kKTAhead steps, late(i) issues the i-th operand read of the dq product
// that follows.
template <typename Load, typename Valu, typename Late, typename Pre>
__device__ __forceinline__ void scores_dp(const char* Ks, const char* Vs, const bf16x8* qreg,
                                          const bf16x8* dreg, const TileOffsets& o, f32x16& s,
                                          f32x16& dp, Load&& load, Valu&& valu, Late&& late,
                                          Pre&& pre) {
  bf16x8 kr[16], vr[16];
#pragma unroll
  for (int i = 0; i < kSDAhead; ++i) {
    kr[i] = tile_row16(Ks, o, i);
    vr[i] = tile_row16(Vs, o, i);
  }
  mfma_fence();
  pre();
  s = zero16();
  dp = zero16();
#pragma unroll
  for (int ks = 0; ks < 16; ++ks) {
    if (ks + kSDAhead < 16) {
      kr[ks + kSDAhead] = tile_row16(Ks, o, ks + kSDAhead);
      vr[ks + kSDAhead] = tile_row16(Vs, o, ks + kSDAhead);
    }
    s = mfma32(kr[ks], qreg[ks], s);
    dp = mfma32(vr[ks], dreg[ks], dp);
    if (ks < 8) load(ks);
    valu(ks);
    if (ks >= 16 - kKTAhead) late(ks - (16 - kKTAhead));
    mfma_fence();
  }
}

// dq^T += K^T dS^T for one 32-key tile; dS register block kk holds keys
// 16kk + {4h..4h+3, 8+4h..8+4h+3}, matched by the transposed K reads.
// Operand i is dims block i/2, key half i%2.
__device__ __forceinline__ bf16x8 dq_kt(const char* Ks, const TileOffsets& o, int i) {
  return (i & 1) ? tile_col8(Ks, o, i >> 1, 16, 24) : tile_col8(Ks, o, i >> 1, 0, 8);
}
// kt0: the first kKTAhead operands, already read (or null: read them here).
// kDefer > 0: the last kDefer MFMAs are left to `tail` (operands and dS).
template <int kDefer = 0>
__device__ __forceinline__ void dq_update(const char* Ks, const bf16x8& d0, const bf16x8& d1,
                                          f32x16* acc, const TileOffsets& o,
                                          const bf16x8* kt0 = nullptr, DqTail* tail = nullptr) {
  bf16x8 kt[16];
  auto read = [&](int i) { return dq_kt(Ks, o, i); };
#pragma unroll
  for (int i = 0; i < kKTAhead; ++i) kt[i] = kt0 ? kt0[i] : read(i);
#pragma unroll
  for (int i = 0; i < 16 - kDefer; ++i) {
    if (i + kKTAhead < 16) kt[i + kKTAhead] = read(i + kKTAhead);
    acc[i >> 1] = mfma32(kt[i], (i & 1) ? d1 : d0, acc[i >> 1]);
    mfma_fence();
  }
  if constexpr (kDefer > 0) {
#pragma unroll
    for (int j = 0; j < kDefer; ++j) tail->kt[j] = kt[16 - kDefer + j];
    tail->d0 = d0;
    tail->d1 = d1;
  }
}

// dS = P (dP - Delta) of one tile, P = exp2(s*scale*log2e - lse2) (masked
// keys carry s = -inf, so P = 0), cut into pieces issued between the S/dP
// MFMAs of the next tile: pieces 0-7 two elements each, 8 and 9 the packed
// bf16 operand halves.
struct DsPieces {
  f32x16& s;
  const f32x16& dp;
  float c, lse2, delta;
  bf16x8 d0, d1;
  __device__ __forceinline__ void piece(int k) {
    if (k < 8) {
#pragma unroll
      for (int r = 2 * k; r < 2 * k + 2; ++r)
        s[r] = __builtin_amdgcn_exp2f(fmaf(s[r], c, -lse2)) * (dp[r] - delta);
      // keep the exponentials here (the compiler would sink them to their use)
      asm volatile("" ::"v"(s[2 * k]), "v"(s[2 * k + 1]));
    } else if (k == 8) {
      d0 = pack8(s, 0);
      asm volatile("" ::"v"(d0));
    } else if (k == 9) {
      d1 = pack8(s, 1);
      asm volatile("" ::"v"(d1));
    }
  }
  __device__ __forceinline__ void all() {
#pragma unroll
    for (int k = 0; k < 10; ++k) piece(k);
  }
};

// One pipelined step: S^T and dP^T of the tile in `cur`, with dS of the
// previous tile (s_prev / dp_prev) computed between their MFMAs, then that
// tile's dq product (K in `prev_k`).  Ring slots are distinct (see the forward
// kernel).  `pe` holds the page-table entry of t0_next on entry and that of
// t0_after on return.  This tile's masked scores and dP go to s_out / dp_out,
// a register set other than s_prev / dp_prev: the loop alternates two sets, so
// no step copies its results into place.
template <PageForm kForm, bool kFirst>
__device__ __forceinline__ void dq_step(const BwdArgs& a, char* __restrict__ next,
                                        const char* __restrict__ cur,
                                        const char* __restrict__ prev_k, const TileFetch& kf,
                                        const TileFetch& vf, const PageLookup& pl, int32_t& pe,
                                        int64_t t0_next, int64_t t0_after, int64_t k_hi,
                                        int64_t t0, int64_t kb, int64_t k_all, int64_t my_lim,
                                        int w, const bf16x8* qreg, const bf16x8* dreg,
                                        const TileOffsets& to, int hh, float lse2, float delta,
                                        f32x16* acc, f32x16& s_prev, f32x16& dp_prev,
                                        f32x16& s, f32x16& dp, DqTail& tail) {
  DsPieces ds{s_prev, dp_prev, a.scale_log2, lse2, delta};
  // the deferred end of the dq product two tiles back (zeros before the
  // first); the per-key variant (short pages) has no registers to carry it
  auto pre = [&]() {
    if constexpr (kForm != kRowPage) {
      if (!kFirst) tail.run(acc);
    }
  };
  auto valu = [&](int k) {
    if (!kFirst) ds.piece(k);
  };
  constexpr bool kEarly = LS_DQ_KT_EARLY && !kFirst;
  bf16x8 kt0[kKTAhead];
  auto late = [&](int i) {
    if (kEarly) kt0[i] = dq_kt(prev_k, to, i);
  };
  if (kForm == kRowPage) {
    kf.issue_rows(next, a.page_table, a.log2_page, t0_next, k_hi);
    vf.issue_rows(next + kTileBytes, a.page_table, a.log2_page, t0_next, k_hi);
    scores_dp(cur, cur + kTileBytes, qreg, dreg, to, s, dp, [](int) {}, valu, late, pre);
  } else {
    const int64_t pos_next = TileFetch::lookup_pos<kForm>(t0_next, k_hi, w);
    const int64_t prow_next = pl.row(pe, pos_next);
    pe = pl.load(TileFetch::lookup_pos<kForm>(t0_after, k_hi, w));
    // the entry load stays ahead of the stage's loads; scalar and vector ALU
    // work may cross, so the next stage's descriptors are built among the MFMAs
    __builtin_amdgcn_sched_barrier(0x0006);
    const __amdgpu_buffer_rsrc_t rk = kf.page_rsrc(prow_next), rv = vf.page_rsrc(prow_next);
    const int nv = (int)min(k_hi - pos_next, (int64_t)kQBN);
    scores_dp(cur, cur + kTileBytes, qreg, dreg, to, s, dp, [&](int i) {
      if (i < 4) kf.issue_one_u24(next, rk, i, nv);
      else vf.issue_one_u24(next + kTileBytes, rv, i - 4, nv);
    }, valu, late, pre);
  }
  if (t0 < kb || t0 + kQBN > k_all) mask_keys(s, t0, kb, my_lim, hh);
  if (!kFirst)
    dq_update<kForm == kRowPage ? 0 : kDqDefer>(prev_k, ds.d0, ds.d1, acc, to,
                                                kEarly ? kt0 : nullptr, &tail);
}

// Workgroup z works on a chunk of one of the key ranges.  With `part` each writes
// its unscaled sums to part[z] and dq_reduce_kernel adds them in order; without,
// there is one range in one chunk.  Under a tail (DqRanges) the row tiles before
// tail_x write their chunks first, or their result where they have one chunk, and
// the tail's chunks follow, [chunk][token past the first of tail_x].
template <PageForm kForm>
__global__ __launch_bounds__(256, 1) void bwd_dq_bf16_d256_kernel(BwdArgs a, DqRanges ranges,
                                                                  float* __restrict__ part) {
  __shared__ __attribute__((aligned(1024))) char smem[kQSlots * kQStage];

  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform (scalar)
  const int l32 = lane & 31, hh = lane >> 5;
  const int lg = a.log2_group;
  const int rows_total = a.n_q << lg;
  WorkItem wi;
  int64_t slice = 0;          // the partial sums' place: slice * n_q_heads rows, tokens from tok0
  int tok0 = 0;
  bool direct = !part, tail_rows = false;
  if (ranges.tail_chunks == 0) {
#if LS_XCD_MAP
    wi = xcd_work_item();
#else
    wi = WorkItem{(int)blockIdx.x, (int)blockIdx.y, (int)blockIdx.z};
#endif
    slice = (int64_t)wi.z * a.n_q;
  } else {
    const uint32_t head_x = ranges.tail_x, tail_x = (rows_total + kQBM - 1) / kQBM - head_x;
    const uint32_t ny = a.n_kv_heads, n_head = head_x * ny * ranges.z0[1];
    uint32_t w = tail_spread(blockIdx.x, gridDim.x, n_head);
    const int split = (int)(head_x * kQBM) >> lg;   // first token of the tail
    tail_rows = w >= n_head;
    if (tail_rows) w -= n_head;
    const uint32_t nx = tail_rows ? tail_x : head_x;
    wi.x = (int)(w % nx + (tail_rows ? head_x : 0));
    wi.y = (int)((w / nx) % ny);
    wi.z = (int)(w / (nx * ny));
    direct = !tail_rows && ranges.z0[1] == 1;
    if (tail_rows) {
      tok0 = split;
      slice = (ranges.z0[1] > 1 ? (int64_t)ranges.z0[1] * split : 0) +
              (int64_t)wi.z * (a.n_q - split);
    } else {
      slice = (int64_t)wi.z * split;
    }
  }
  const int g = wi.y;
  const int row0 = wi.x * kQBM;
  const int prow = row0 + w * 32 + l32;
  const bool row_ok = prow < rows_total;
  const int tok = prow >> lg;
  const int head = (g << lg) + (prow & ((1 << lg) - 1));
  const int tok_first = row0 >> lg;
  const int tok_last = min(a.n_q - 1, (row0 + kQBM - 1) >> lg);
  const int ri = tail_rows ? 0 : ranges.of(wi.z);
  const int64_t kv_begin = ranges.begin[ri];
  const int64_t chunk_keys = (int64_t)(tail_rows ? ranges.tail_per : ranges.per[ri]) * kQBN;
  const int64_t c_lo = (kv_begin & ~int64_t(kQBN - 1)) + (wi.z - ranges.z0[ri]) * chunk_keys;
  const int64_t kb = max(kv_begin, c_lo);
  const int64_t ke = min(ranges.end[ri], c_lo + chunk_keys);
  const int64_t k_hi = min(ke, a.q_pos0 + tok_last + 1);
  const int64_t k_all = min(ke, a.q_pos0 + tok_first + 1);
  const int64_t my_lim = min(ke, a.q_pos0 + tok + 1);
  const int64_t k_lo = kb & ~int64_t(kQBN - 1);
  const int n_tiles = k_hi > kb ? (int)((k_hi - k_lo + kQBN - 1) / kQBN) : 0;

  const bool add = direct && a.accumulate_dq;
  float* dq = direct ? a.dq + ((int64_t)tok * a.n_q_heads + head) * kD
                     : part + ((slice + tok - tok0) * a.n_q_heads + head) * kD;
  if (n_tiles == 0) {
    if (row_ok && !add) {
      const f32x4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int c = 0; c < 32; ++c) *reinterpret_cast<f32x4*>(dq + c * 8 + hh * 4) = z;
    }
    return;
  }

  TileFetch kf, vf;
  kf.init<kForm>(static_cast<const __bf16*>(a.k_pool) + (int64_t)g * kD, a.k_pos_stride, lane, w);
  vf.init<kForm>(static_cast<const __bf16*>(a.v_pool) + (int64_t)g * kD, a.v_pos_stride, lane, w);
  PageLookup pl;
  pl.init(a.page_table, a.log2_page);
  const TileOffsets to = tile_offsets(lane);
  // tiles past the last one are clamped to it (refetched into an unread slot),
  // so every iteration issues exactly one stage of direct loads
  auto clamp = [&](int t) { return t < n_tiles ? t : n_tiles - 1; };
#pragma unroll
  for (int i = 0; i < kQAhead; ++i) {
    const int64_t t0 = k_lo + (int64_t)clamp(i) * kQBN;
    char* st = smem + i * kQStage;
    const int64_t pos = TileFetch::lookup_pos<kForm>(t0, k_hi, w);
    const int64_t pr = kForm == kRowPage ? 0 : phys_pos_uniform(a.page_table, pos, a.log2_page);
    kf.issue<kForm>(st, a.page_table, a.log2_page, t0, k_hi, pos, pr);
    vf.issue<kForm>(st + kTileBytes, a.page_table, a.log2_page, t0, k_hi, pos, pr);
  }
  auto tile0 = [&](int t) { return k_lo + (int64_t)clamp(t) * kQBN; };
  int32_t pe = kForm == kRowPage
                   ? 0 : pl.load(TileFetch::lookup_pos<kForm>(tile0(kQAhead), k_hi, w));

  bf16x8 qreg[16], dreg[16];
  {
    const int64_t rh = (int64_t)tok * a.n_q_heads + head;
    const __bf16* qrow = static_cast<const __bf16*>(a.q) + rh * kD + hh * 8;
    const __bf16* drow = static_cast<const __bf16*>(a.d_out) + rh * kD + hh * 8;
#pragma unroll
    for (int ks = 0; ks < 16; ++ks) {
      if (row_ok) {
        qreg[ks] = *reinterpret_cast<const bf16x8*>(qrow + ks * 16);
        dreg[ks] = *reinterpret_cast<const bf16x8*>(drow + ks * 16);
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) qreg[ks][e] = dreg[ks][e] = (__bf16)0.f;
      }
    }
  }
  const int64_t stat = (int64_t)head * a.n_q + (row_ok ? tok : 0);
  const float lse2 = row_ok ? a.lse2[stat] : INFINITY;
  const float delta = row_ok ? a.delta[stat] : 0.f;

  f32x16 acc[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) acc[i] = zero16();
  // masked scores and dP of a tile, in two sets that the steps alternate
  f32x16 s_a, dp_a, s_b, dp_b;
  DqTail tail;
#pragma unroll
  for (int j = 0; j < (kDqDefer > 0 ? kDqDefer : 1); ++j)
#pragma unroll
    for (int e = 0; e < 8; ++e) tail.kt[j][e] = (__bf16)0.f;
  tail.d0 = tail.kt[0];
  tail.d1 = tail.kt[0];
  auto end_step = [&]() {
    wait_vmcnt<(kQAhead - 1) * 8>();
    __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0): the step's LDS reads have landed
    tile_barrier();
  };

  // (a full wait here: the Q/dO loads may have been scheduled after the stages)
  wait_fetch();
  tile_barrier();
  // Iteration t fetches tile t + kQAhead and, before its barrier, waits for
  // the loads of tile t + 1.  Tile t's scores land in set a for even t and in
  // set b for odd t.
  {
    dq_step<kForm, true>(a, smem + kQAhead * kQStage, smem, smem, kf, vf, pl, pe, tile0(kQAhead),
                           tile0(kQAhead + 1), k_hi, k_lo, kb, k_all, my_lim, w, qreg, dreg, to, hh,
                           lse2, delta, acc, s_b, dp_b, s_a, dp_a, tail);
    end_step();
  }
  auto step = [&](int t, f32x16& s_in, f32x16& dp_in, f32x16& s_out, f32x16& dp_out) {
    const int64_t t0 = k_lo + (int64_t)t * kQBN;
    dq_step<kForm, false>(a, smem + ((t + kQAhead) % kQSlots) * kQStage,
                            smem + (t % kQSlots) * kQStage, smem + ((t - 1) % kQSlots) * kQStage,
                            kf, vf, pl, pe, tile0(t + kQAhead), tile0(t + kQAhead + 1), k_hi, t0,
                            kb, k_all, my_lim, w, qreg, dreg, to, hh, lse2, delta, acc, s_in, dp_in,
                            s_out, dp_out, tail);
    end_step();
  };
  int t = 1;
  for (; t + 1 < n_tiles; t += 2) {
    step(t, s_a, dp_a, s_b, dp_b);
    step(t + 1, s_b, dp_b, s_a, dp_a);
  }
  // the last tile's dS and dq product (its scores are in set b when a tile
  // was left over for one more step, else in set a)
  auto finish = [&](f32x16& s_last, f32x16& dp_last) {
    if constexpr (kForm != kRowPage) tail.run(acc);
    DsPieces ds{s_last, dp_last, a.scale_log2, lse2, delta};
    ds.all();
    dq_update(smem + ((n_tiles - 1) % kQSlots) * kQStage, ds.d0, ds.d1, acc, to);
  };
  if (t < n_tiles) {
    step(t, s_a, dp_a, s_b, dp_b);
    finish(s_b, dp_b);
  } else {
    finish(s_a, dp_a);
  }
  wait_fetch();   // no direct load is left in flight when the waves end

  if (row_ok) {
    const float c = direct ? a.scale : 1.f;
#pragma unroll
    for (int db = 0; db < 8; ++db) {
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        f32x4* dst = reinterpret_cast<f32x4*>(dq + 32 * db + 8 * q4 + 4 * hh);
        // (one rounding where it is added, as in dq_reduce_kernel)
        f32x4 v;
        if (add) {
          const f32x4 old = *dst;
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = fmaf(acc[db][4 * q4 + e], c, old[e]);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = acc[db][4 * q4 + e] * c;
        }
        *dst = v;
      }
    }
  }
}

// ============================================================== dk/dv kernel
// Workgroup = 4 waves = kKeysPerWG response keys of one KV head (wave w owns
// keys j0 + 32w .. +31; lane l owns key l % 32 and keeps its K and V rows in
// registers) x one chunk of a.dkdv_rows packed query rows (dkdv_row_chunks).  The chunk's 32-row
// tiles of Q and dO stream into a four-slot LDS ring by direct loads, two
// tiles ahead, each with the rows' lse * log2(e) and Delta.  Per tile:
//   S = Q K^T, dP = dO V^T (lane = key, result registers = rows),
//   P = exp2(S * scale * log2(e) - lse2), dS = P (dP - Delta), zero where the
//   row does not see the key (causal edge) or lies past the last row,
//   dv^T += dO^T P, dk^T += Q^T dS (transposed reads of the row tiles).
// The chunk's partial sums go to the workspace; dkdv_reduce_kernel adds the
// active chunks in order (deterministic), scales dk and writes or accumulates.
constexpr int kKeysPerWG = kDkdvKeys;
constexpr int kRStat = 256;                                // per wave: 32 lse2 + 32 Delta floats
constexpr int kRStage = 2 * kTileBytes + 4 * kRStat;       // Q tile, dO tile, stats
constexpr int kRAhead = 2;
constexpr int kRSlots = kRAhead + 2;

// First row (a multiple of 32) of `chunk` that can see a key of the block
// starting at j0 (rows of tokens >= j0 - q_pos0); the chunk is active when it
// is below the chunk's end.  Shared by the dk/dv and reduce kernels.
__device__ __forceinline__ int dkdv_row_lo(const BwdArgs& a, int64_t j0, int chunk) {
  int64_t first_tok = j0 - a.q_pos0;
  if (first_tok < 0) first_tok = 0;
  const int64_t rows_total = (int64_t)a.n_q << a.log2_group;
  const int64_t vis = min(rows_total, first_tok << a.log2_group) & ~int64_t(31);
  return (int)max((int64_t)chunk * a.dkdv_rows, vis);
}
__device__ __forceinline__ int dkdv_row_hi(const BwdArgs& a, int chunk) {
  return (int)min((int64_t)a.n_q << a.log2_group, (int64_t)(chunk + 1) * a.dkdv_rows);
}

// Direct loads of 32 packed query rows (token, head of KV group g) of Q or dO
// into a row tile (same swizzled layout and lane mapping as the key tiles);
// rows at or beyond rows_total repeat the last row.
struct RowFetch {
  int lane_off[4], lds_row[4], lane_row[4];
  __device__ __forceinline__ void init(int lane, int w) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      lds_row[i] = 8 * w + 2 * i;
      lane_row[i] = lds_row[i] + (lane >> 5);
      lane_off[i] = ((lane & 31) ^ tile_swz(lane_row[i])) * 16;
    }
  }
  // byte offset of instruction i's row for tile row row0 in a [n_q, Hq, 256] bf16 array
  __device__ __forceinline__ int offset(const BwdArgs& a, int g, int row0, int rows_total,
                                        int i) const {
    const int prow = min(row0 + lane_row[i], rows_total - 1);
    const int head = (g << a.log2_group) + (prow & ((1 << a.log2_group) - 1));
    return ((prow >> a.log2_group) * a.n_q_heads + head) * kRowBytes + lane_off[i];
  }
  __device__ __forceinline__ void issue_one(char* tile, __amdgpu_buffer_rsrc_t r, int off,
                                            int i) const {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, LS_LDS(tile + lds_row[i] * kTileRow), 16, off, 0, 0,
                                             0);
  }
};

__global__ __launch_bounds__(256, 1) void bwd_dkdv_bf16_d256_kernel(BwdArgs a, int64_t key0,
                                                                   int64_t key_end) {
  __shared__ __attribute__((aligned(1024))) char smem[kRSlots * kRStage];

  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hh = lane >> 5;
  const int g = blockIdx.y, chunk = blockIdx.z;
  const int lg = a.log2_group;
  const int rows_total = a.n_q << lg;
  const int64_t j0 = key0 + (int64_t)blockIdx.x * kKeysPerWG;
  const int64_t jw = j0 + 32 * w;          // first key of this wave
  const int64_t j_mine = jw + l32;
  const int row_lo = dkdv_row_lo(a, j0, chunk);
  const int row_hi = dkdv_row_hi(a, chunk);
  if (row_lo >= row_hi) return;            // no row of the chunk sees a key of the block
  const int n_tiles = (row_hi - row_lo + 31) / 32;

  // K and V rows of this lane's key (B operands: lane = key, 8 dims per step)
  bf16x8 kreg[16], vreg[16];
  {
    const bool ok = j_mine < key_end;
    const int64_t pr = ok ? phys_pos(a.page_table, j_mine, a.log2_page) : 0;
    const __bf16* kr = static_cast<const __bf16*>(a.k_pool) + pr * a.k_pos_stride + g * kD + hh * 8;
    const __bf16* vr = static_cast<const __bf16*>(a.v_pool) + pr * a.v_pos_stride + g * kD + hh * 8;
#pragma unroll
    for (int ks = 0; ks < 16; ++ks) {
      if (ok) {
        kreg[ks] = *reinterpret_cast<const bf16x8*>(kr + ks * 16);
        vreg[ks] = *reinterpret_cast<const bf16x8*>(vr + ks * 16);
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) kreg[ks][e] = vreg[ks][e] = (__bf16)0.f;
      }
    }
  }

  const __amdgpu_buffer_rsrc_t rq = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<void*>(a.q), (short)0, 0x7FFFFFFF, 0x00020000);
  const __amdgpu_buffer_rsrc_t rd = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<void*>(a.d_out), (short)0, 0x7FFFFFFF, 0x00020000);
  // Delta and lse2 live in one workspace block; lanes 0-31 load lse2 rows, 32-63 Delta rows
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float*>(a.delta), (short)0, 0x7FFFFFFF, 0x00020000);
  const int lse2_off = (int)((const char*)a.lse2 - (const char*)a.delta);
  RowFetch rf;
  rf.init(lane, w);
  auto clamp = [&](int t) { return t < n_tiles ? t : n_tiles - 1; };
  auto stats = [&](char* st, int row0) {
    const int prow = min(row0 + l32, rows_total - 1);
    const int head = (g << lg) + (prow & ((1 << lg) - 1));
    const int off = (hh ? 0 : lse2_off) + (head * a.n_q + (prow >> lg)) * 4;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, LS_LDS(st + 2 * kTileBytes + kRStat * w), 4, off,
                                             0, 0, 0);
  };
  auto fetch = [&](char* st, int row0, int i) {   // instruction i of a stage's row loads
    const int off = rf.offset(a, g, row0, rows_total, i & 3);
    if (i < 4) rf.issue_one(st, rq, off, i);
    else rf.issue_one(st + kTileBytes, rd, off, i - 4);
  };
#pragma unroll
  for (int i = 0; i < kRAhead; ++i) {
    char* st = smem + i * kRStage;
    const int row0 = row_lo + 32 * clamp(i);
    stats(st, row0);
#pragma unroll
    for (int k = 0; k < 8; ++k) fetch(st, row0, k);
  }
  const TileOffsets to = tile_offsets(lane);
  f32x16 dk[8], dv[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) dk[i] = dv[i] = zero16();
  wait_fetch();
  tile_barrier();

  for (int t = 0; t < n_tiles; ++t) {
    char* cur = smem + (t % kRSlots) * kRStage;
    char* next = smem + ((t + kRAhead) % kRSlots) * kRStage;
    const int row_next = row_lo + 32 * clamp(t + kRAhead);
    stats(next, row_next);
    __builtin_amdgcn_sched_barrier(0);
    f32x16 s, dp;
    scores_dp(cur, cur + kTileBytes, kreg, vreg, to, s, dp,
              [&](int i) { fetch(next, row_next, i); }, [](int) {}, [](int) {}, [] {});
    const float* st = reinterpret_cast<const float*>(cur + 2 * kTileBytes + kRStat * w);
    const int row0 = row_lo + 32 * t;
    const bool edge = a.q_pos0 + (row0 >> lg) < jw + 31 || row0 + 32 > rows_total;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const f32x4 l2 = *reinterpret_cast<const f32x4*>(st + 8 * m + 4 * hh);
      const f32x4 dl = *reinterpret_cast<const f32x4*>(st + 32 + 8 * m + 4 * hh);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = 4 * m + e;
        float p = __builtin_amdgcn_exp2f(fmaf(s[r], a.scale_log2, -l2[e]));
        if (edge) {
          const int row = row0 + acc_key(r, hh);
          if (row >= rows_total || a.q_pos0 + (row >> lg) < j_mine) p = 0.f;
        }
        s[r] = p;
        dp[r] = p * (dp[r] - dl[e]);
      }
    }
    dq_update(cur + kTileBytes, pack8(s, 0), pack8(s, 1), dv, to);   // dv^T += dO^T P
    dq_update(cur, pack8(dp, 0), pack8(dp, 1), dk, to);              // dk^T += Q^T dS
    __builtin_amdgcn_s_waitcnt(0x0F79);   // vmcnt(9): only the newest stage may be in flight
    tile_barrier();
  }
  wait_fetch();

  // partial sums of this chunk: part[chunk][0 = dk, 1 = dv][g][key - key0][256]
  if (j_mine < key_end) {
    const int64_t n_part = key_end - key0;
    const int64_t kidx = j_mine - key0;
    float* pk = a.dkdv_part + (((int64_t)chunk * 2 * a.n_kv_heads + g) * n_part + kidx) * kD;
    float* pv = pk + (int64_t)a.n_kv_heads * n_part * kD;
#pragma unroll
    for (int db = 0; db < 8; ++db) {
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const int d0 = 32 * db + 8 * q4 + 4 * hh;
        f32x4 kv, vv;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          kv[e] = dk[db][4 * q4 + e];
          vv[e] = dv[db][4 * q4 + e];
        }
        *reinterpret_cast<f32x4*>(pk + d0) = kv;
        *reinterpret_cast<f32x4*>(pv + d0) = vv;
      }
    }
  }
}

// dk_resp / dv_resp for keys [key0, key_end): the sum over the active row
// chunks, in chunk order; dk is scaled by softmax_scale.  Thread = 4 dims of
// one key of one KV head.
__global__ __launch_bounds__(256) void dkdv_reduce_kernel(BwdArgs a, int64_t key0, int64_t key_end,
                                                          int n_chunks) {
  const int64_t n_keys = key_end - key0;
  const int64_t item = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;   // (key, g, d4)
  if (item >= n_keys * a.n_kv_heads * (kD / 4)) return;
  const int d0 = (int)(item % (kD / 4)) * 4;
  const int g = (int)((item / (kD / 4)) % a.n_kv_heads);
  const int64_t j = key0 + item / ((kD / 4) * a.n_kv_heads);
  const int64_t j0 = key0 + (j - key0) / kKeysPerWG * kKeysPerWG;
  f32x4 sk = {0.f, 0.f, 0.f, 0.f}, sv = sk;
  for (int c = 0; c < n_chunks; ++c) {
    if (dkdv_row_lo(a, j0, c) >= dkdv_row_hi(a, c)) continue;
    const float* pk =
        a.dkdv_part + (((int64_t)c * 2 * a.n_kv_heads + g) * n_keys + j - key0) * kD + d0;
    sk += *reinterpret_cast<const f32x4*>(pk);
    sv += *reinterpret_cast<const f32x4*>(pk + (int64_t)a.n_kv_heads * n_keys * kD);
  }
  sk *= a.scale;
  const int64_t r = ((j - a.prefix_len) * a.n_kv_heads + g) * kD + d0;
  f32x4* dkr = reinterpret_cast<f32x4*>(a.dk_resp + r);
  f32x4* dvr = reinterpret_cast<f32x4*>(a.dv_resp + r);
  if (a.accumulate_dkv) {
    sk += *dkr;
    sv += *dvr;
  }
  *dkr = sk;
  *dvr = sv;
}

}  // namespace

namespace {

// Key chunks of a dq launch.  One workgroup (128 KiB of LDS) runs per CU, so
// `items` workgroups of `tiles` key tiles take ceil(items / 256) rounds of
// (tiles + 6) tile times: 6 for the first loads, the Q and dO rows and the
// result.  c chunks cut the rounds to whole shares of fewer tiles (10 items
// leave 246 CUs idle, 140 leave 116) and add the partial sums' way through
// memory, about 4.7e-4 tile times per row and chunk (1 KiB out and back in
// against 32 KiB of K and V per 0.95 us) and a launch.  The chunk counts that
// fill 1 to 8 rounds are priced, and within each the one that balances tiles
// and partial sums, if smaller; one chunk where nothing is less (512 items: 2
// rounds either way).  Measured: 77 rows x 16 heads over 32,768 keys 836 -> 76 us
// (25 chunks), 1,111 rows over 12,500 keys 396 -> 345 us (3 chunks), 952 rows
// over 32,768 keys 952 -> 568 us (2 chunks), the reduce included.
int dq_chunks(const BwdArgs& a, int64_t items, int64_t tiles) {
  const double rows = (double)a.n_q * a.n_q_heads;
  const int64_t most = std::min<int64_t>({dq_part_rows(a.n_q, a.group) / ((int64_t)a.n_q * a.n_q_heads),
                                          256, tiles / 4});
  int best = 1;
  double least = (double)((items + 255) / 256) * (double)(tiles + 6);
  for (int k = 1; k <= 8; ++k) {
    const int64_t fill = 256 * k / items;
    const int64_t balance = (int64_t)sqrt((double)k * (double)tiles / (4.7e-4 * rows)) + 1;
    const int64_t c = std::min({fill, balance, most});
    if (c < 2) continue;
    const double cost = (double)((items * c + 255) / 256) * (double)((tiles + c - 1) / c + 6) + 5 +
                        4.7e-4 * rows * (double)c;
    if (cost < least) {
      best = (int)c;
      least = cost;
    }
  }
  return best;
}

// Time of n workgroups of `t` tile times on 256 CUs.  The last round's CUs clock
// higher where fewer are busy (214 of 256: 1.18 us a tile instead of 1.32; 164:
// 0.92 of 1.19; 96: 0.90).
double rounds(int64_t n, double t) {
  const double f = (double)(n % 256) / 256;
  return t * ((double)(n / 256) + (f > 0 ? std::max(0.75, 0.36 + 0.64 * f) : 0.));
}

// A tail for a range of `chunks` chunks, where that is faster: the row tiles that
// fill whole rounds keep few chunks, and those left over share one round among
// all CUs in many, so that no round is nearly empty, within the same room for
// partial sums (chunks of every row would need more: 258 items have room for
// one).  Measured, one range of 204,800 keys, 16 heads on 2: 1,111 tokens (140
// items) 5.35 -> 4.70 ms, 1,536 (192) 7.21 -> 6.43, 2,064 (258) 15.3 -> 8.6, 3,000
// (376) 14.5 -> 12.5: 1,190-1,210 TFLOP/s, as 2,048 and 4,096 tokens reach.
void plan_tail(const BwdArgs& a, int64_t tiles, DqPlan& p) {
  const int64_t nx = ((int64_t)a.n_q * a.group + kQBM - 1) / kQBM, H = a.n_kv_heads;
  const int64_t room = dq_part_rows(a.n_q, a.group) / a.n_q_heads;   // tokens
  const double per_tok = 4.7e-4 * a.n_q_heads;
  auto chunk = [&](int64_t c) { return (tiles + c - 1) / c; };
  double least = 0.98 * (rounds(nx * H * p.chunks, (double)p.per + 6) +
                         (p.chunks > 1 ? 5 + per_tok * a.n_q * p.chunks : 0.));
  for (int64_t c1 = 1; c1 <= 4; ++c1) {
    const int64_t hx = nx * H * c1 / 256 * 256 / (c1 * H);
    if (hx == 0 || hx >= nx) continue;
    const int64_t tok = hx * kQBM / a.group, parts = c1 > 1 ? c1 * tok : 0;
    for (int64_t f = 1; f <= 4; f *= 2) {
      const int64_t c2 = std::min({256 / ((nx - hx) * H * f), tiles / 4,
                                   (room - parts) / (a.n_q - tok)});
      if (c2 < 2) break;
      const int64_t sums = parts + c2 * (a.n_q - tok);
      const double cost = rounds(hx * H * c1, (double)chunk(c1) + 6) +
                          rounds((nx - hx) * H * c2, (double)chunk(c2) + 6) + 5 +
                          (c1 > 1 ? 5 : 0) + per_tok * (double)sums;
      if (cost >= least) continue;
      least = cost;
      p.per = (int32_t)chunk(c1);
      p.chunks = (int32_t)((tiles + p.per - 1) / p.per);
      p.tail_x = (int32_t)hx;
      p.tail_per = (int32_t)chunk(c2);
      p.tail_chunks = (int32_t)((tiles + p.tail_per - 1) / p.tail_per);
    }
  }
}

}  // namespace

DqPlan plan_dq_bf16_d256(const BwdArgs& a, int64_t begin, int64_t end) {
  const int64_t items = ((int64_t)a.n_q * a.group + kQBM - 1) / kQBM * a.n_kv_heads;
  const int64_t tiles = (end - (begin & ~int64_t(kQBN - 1)) + kQBN - 1) / kQBN;
  const int want = dq_chunks(a, items, tiles);
  const int per = (int)((tiles + want - 1) / want);
  const int chunks = (int)((tiles + per - 1) / per);
  // Ranges of no more than one round of workgroups share launches: without the
  // gaps and ragged ends between them, 10 tokens over 8 ranges of 625 keys 166 ->
  // 49 us, 77 over 8 of 32,768 634 -> 577, 952 over the same 5,183 -> 5,116.  A
  // range of several rounds keeps its own, so that the row tiles that share keys
  // stay together (1,111 tokens, 8 ranges of 12,500: 2,731 us apart, 2,825 joined),
  // and one whose single chunk fills half the chip writes its result itself.
  const int64_t wgs = items * chunks;
  DqPlan p{begin, end, chunks, per, 0, wgs <= 256 && (chunks > 1 || wgs < 128)};
  if (!p.joins) plan_tail(a, tiles, p);
  return p;
}

hipError_t launch_dq_bf16_d256(const BwdArgs& a, const DqRanges& r, float* part,
                               hipStream_t stream) {
  const unsigned nx = (unsigned)(((int64_t)a.n_q * a.group + kQBM - 1) / kQBM);
  const dim3 grid = r.tail_chunks == 0
                        ? dim3(nx, a.n_kv_heads, r.z0[r.n])
                        : dim3(a.n_kv_heads * ((unsigned)r.tail_x * r.z0[1] +
                                               (nx - r.tail_x) * r.tail_chunks));
  // (pages of 8 and 16 rows: 2,336 -> 1,962 us per shard with the lookup per wave
  // instead of per row, 2,048 rows x 50,000 keys, as with longer pages)
  switch (page_form(a.log2_page)) {
    case kTilePage:
      hipLaunchKernelGGL(bwd_dq_bf16_d256_kernel<kTilePage>, grid, dim3(256), 0, stream, a, r, part);
      break;
    case kWavePage:
      hipLaunchKernelGGL(bwd_dq_bf16_d256_kernel<kWavePage>, grid, dim3(256), 0, stream, a, r, part);
      break;
    case kRowPage:
      hipLaunchKernelGGL(bwd_dq_bf16_d256_kernel<kRowPage>, grid, dim3(256), 0, stream, a, r, part);
      break;
  }
  return hipGetLastError();
}

hipError_t launch_dkdv_bf16_d256(const BwdArgs& args, int64_t key0, hipStream_t stream) {
  BwdArgs a = args;
  const int64_t n_keys = a.kv_end - key0, packed = (int64_t)a.n_q * a.group;
  const unsigned blocks = (unsigned)((n_keys + kKeysPerWG - 1) / kKeysPerWG);
  const int64_t want = dkdv_launch_chunks(a.n_q, a.group, a.n_kv_heads, n_keys);
  a.dkdv_rows = (int32_t)(((packed + want - 1) / want + 31) / 32 * 32);
  const int n_chunks = (int)((packed + a.dkdv_rows - 1) / a.dkdv_rows);
  hipLaunchKernelGGL(bwd_dkdv_bf16_d256_kernel, dim3(blocks, a.n_kv_heads, n_chunks), dim3(256), 0,
                     stream, a, key0, a.kv_end);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int64_t items = n_keys * a.n_kv_heads * (kD / 4);
  hipLaunchKernelGGL(dkdv_reduce_kernel, dim3((unsigned)((items + 255) / 256)), dim3(256), 0,
                     stream, a, key0, a.kv_end, n_chunks);
  return hipGetLastError();
}

}  // namespace ls
