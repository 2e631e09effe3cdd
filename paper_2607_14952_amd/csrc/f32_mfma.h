// Shared pieces of the fp32 matrix-core kernels (v_mfma_f32_32x32x2_f32).
//
// Operand layout of the 32x32x2 instruction: lane l = 32h + j gives A[j][h] and
// B[h][j]; D register r of lane l is row 8(r/4) + 4h + r%4, column j.  A 32x32
// product over the head dimensions lets lane half h take dimensions
// h*kDP/2 .. h*kDP/2 + kDP/2 - 1 (step t pairs dimensions t and kDP/2 + t), so
// a lane's operand values are contiguous.  A product over the 32 rows of such
// a result pairs, in step r, the rows held by register r of the two lane
// halves: the lane's own register is then the B operand, with no exchange.
//
// Head dimensions are padded with zeros to kDP in {64, 96, 128}; rows are
// moved as 16-byte vectors, so the true widths must be multiples of 4.
#pragma once
#include <math.h>

#include "f32_rows.h"
#include "ls_internal.h"
#include "mfma_common.h"

namespace ls {
namespace f32m {

constexpr int kMaxWidth = 128;

// LDS strides (floats): rows read one per lane (16-byte reads of 16 lanes on
// 16 rows fall in 16 distinct bank groups), and rows read column-wise (the two
// rows of one read, 4 apart, lie 128 bytes apart modulo 256: disjoint banks).
template <int kDP> constexpr int kRowS = kDP + 4;
template <int kDP> constexpr int kColS = kDP + 8;

__device__ __forceinline__ f32x16 mfma(float a, float b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// Row (within a 32-row tile) of result register r in lane half h.
__device__ __forceinline__ int row_of(int r, int h) { return 8 * (r >> 2) + 4 * h + (r & 3); }

// 16-byte piece at column c of a row of d floats: past the row's end the last
// piece is read instead (no branch keeps loads from overlapping), and pad()
// makes it zeros once the value is used.
__device__ __forceinline__ f32x4 load_piece(const float* row, int c, int d) {
  return *reinterpret_cast<const f32x4*>(row + min(c, d - 4));
}
__device__ __forceinline__ f32x4 pad(const f32x4& v, int c, int d) {
  return c < d ? v : f32x4{0.f, 0.f, 0.f, 0.f};
}

// This lane's half of a row of width d: kDP / 2 floats.
template <int kDP>
__device__ __forceinline__ void load_half_row(float* v, const float* row, int d, int h) {
  f32x4 x[kDP / 8];
#pragma unroll
  for (int t = 0; t < kDP / 8; ++t) x[t] = load_piece(row, h * (kDP / 2) + 4 * t, d);
#pragma unroll
  for (int t = 0; t < kDP / 8; ++t) {
    const f32x4 y = pad(x[t], h * (kDP / 2) + 4 * t, d);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[4 * t + e] = y[e];
  }
}

// Operand reads run kAhead steps ahead of the MFMAs that use them (mfma_fence
// keeps them there): an MFMA takes 64 cycles, so a read of the step before
// would still be in flight when it is needed.
constexpr int kAhead = 2;

// 32x32 product of the LDS rows (one per lane, stride kS) with the lane's row,
// in two chains (an MFMA that adds to the result of the one before it waits
// for it).
template <int kDP, int kS>
__device__ __forceinline__ f32x16 row_product(const float* rows, const float* v, int j, int h) {
  constexpr int kSteps = kDP / 8;   // 4 dimensions of each half
  const float* src = rows + j * kS + h * (kDP / 2);
  f32x4 x[kSteps];
#pragma unroll
  for (int t = 0; t < kAhead; ++t) x[t] = *reinterpret_cast<const f32x4*>(src + 4 * t);
  mfma_fence();
  f32x16 s0 = zero16(), s1 = zero16();
#pragma unroll
  for (int t = 0; t < kSteps; ++t) {
    if (t + kAhead < kSteps)
      x[t + kAhead] = *reinterpret_cast<const f32x4*>(src + 4 * (t + kAhead));
    s0 = mfma(x[t][0], v[4 * t], s0);
    s1 = mfma(x[t][1], v[4 * t + 1], s1);
    s0 = mfma(x[t][2], v[4 * t + 2], s0);
    s1 = mfma(x[t][3], v[4 * t + 3], s1);
    mfma_fence();
  }
  return s0 + s1;
}

// Two such products, one chain each, interleaved.
template <int kDP, int kS>
__device__ __forceinline__ void row_products(const float* rows0, const float* v0, f32x16& s0,
                                             const float* rows1, const float* v1, f32x16& s1, int j,
                                             int h) {
  constexpr int kSteps = kDP / 8;
  const int off = j * kS + h * (kDP / 2);
  f32x4 x[kSteps], y[kSteps];
  auto read = [&](int t) {
    x[t] = *reinterpret_cast<const f32x4*>(rows0 + off + 4 * t);
    y[t] = *reinterpret_cast<const f32x4*>(rows1 + off + 4 * t);
  };
#pragma unroll
  for (int t = 0; t < kAhead; ++t) read(t);
  mfma_fence();
  s0 = zero16();
  s1 = zero16();
#pragma unroll
  for (int t = 0; t < kSteps; ++t) {
    if (t + kAhead < kSteps) read(t + kAhead);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      s0 = mfma(x[t][e], v0[4 * t + e], s0);
      s1 = mfma(y[t][e], v1[4 * t + e], s1);
    }
    mfma_fence();
  }
}

// The rows of a 32-row tile, by result register, that lie in [lo, hi) (offsets
// from the tile's first, any value).
__device__ __forceinline__ bool in_rows(int r, int h, int64_t lo, int64_t hi) {
  const int l = (int)min(max(lo, (int64_t)0), (int64_t)32);
  const int u = (int)min(max(hi, (int64_t)0), (int64_t)32);
  return row_of(r, h) >= l && row_of(r, h) < u;
}

// acc (kDP x 32, in blocks of 32 dimensions) += rows^T (32 LDS rows) x p.
template <int kDP, int kS>
__device__ __forceinline__ void col_product(const float* rows, const f32x16& p, f32x16* acc, int j,
                                            int h) {
  constexpr int kDB = kDP / 32;
  const float* src = rows + 4 * h * kS + j;
  float x[16][kDB];
  auto read = [&](int r) {
#pragma unroll
    for (int b = 0; b < kDB; ++b) x[r][b] = src[row_of(r, 0) * kS + 32 * b];
  };
#pragma unroll
  for (int r = 0; r < kAhead; ++r) read(r);
  mfma_fence();
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    if (r + kAhead < 16) read(r + kAhead);
#pragma unroll
    for (int b = 0; b < kDB; ++b) acc[b] = mfma(x[r][b], p[r], acc[b]);
    mfma_fence();
  }
}

// K and V rows of kN consecutive 32-key tiles on their way to LDS: 256 threads
// hold kN * kDP / 32 16-byte pieces of each, loaded while the previous tiles are
// computed, and the page-table entries of the stage after.  Keys outside
// [kb, k_hi) repeat the nearest one inside (the kernels mask them).
template <int kDP, int kN>
struct KvStage {
  static constexpr int kPieces = kN * kDP / 32;
  f32x4 k[kPieces], v[kPieces];
  int32_t page[kPieces];
  __device__ __forceinline__ static int64_t key_pos(int i, int64_t t0, int64_t kb, int64_t k_hi,
                                                    int tid) {
    const int64_t pos = t0 + (tid + 256 * i) / (kDP / 4);
    return min(max(pos, kb), k_hi - 1);
  }
  template <typename Args>
  __device__ __forceinline__ void load_pages(const Args& a, int64_t t0, int64_t kb, int64_t k_hi,
                                             int tid) {
#pragma unroll
    for (int i = 0; i < kPieces; ++i)
      page[i] = a.page_table[key_pos(i, t0, kb, k_hi, tid) >> a.log2_page];
  }
  // rows of the tiles at t0 (whose page entries are here), then the entries of t0 + 32 kN
  template <typename Args>
  __device__ __forceinline__ void load(const Args& a, int g, int64_t t0, int64_t kb, int64_t k_hi,
                                       int tid) {
    const float* kp = static_cast<const float*>(a.k_pool) + (int64_t)g * a.head_dim;
    const float* vp = static_cast<const float*>(a.v_pool) + (int64_t)g * a.head_dim_v;
    const int64_t slot = (int64_t(1) << a.log2_page) - 1;
#pragma unroll
    for (int i = 0; i < kPieces; ++i) {
      const int c = 4 * ((tid + 256 * i) % (kDP / 4));
      const int64_t pr =
          ((int64_t)page[i] << a.log2_page) | (key_pos(i, t0, kb, k_hi, tid) & slot);
      k[i] = load_piece(kp + pr * a.k_pos_stride, c, a.head_dim);
      v[i] = load_piece(vp + pr * a.v_pos_stride, c, a.head_dim_v);
    }
    load_pages(a, t0 + 32 * kN, kb, k_hi, tid);
  }
  template <int kKS, int kVS, typename Args>
  __device__ __forceinline__ void store(const Args& a, float* ks, float* vs, int tid) const {
#pragma unroll
    for (int i = 0; i < kPieces; ++i) {
      const int idx = tid + 256 * i;
      const int key = idx / (kDP / 4), c = 4 * (idx % (kDP / 4));
      *reinterpret_cast<f32x4*>(ks + key * kKS + c) = pad(k[i], c, a.head_dim);
      *reinterpret_cast<f32x4*>(vs + key * kVS + c) = pad(v[i], c, a.head_dim_v);
    }
  }
};

// Accumulator blocks to and from an LDS area of kN x 64 x 16 floats (16-byte
// accesses of consecutive lanes).
template <int kN>
__device__ __forceinline__ void acc_to_lds(float* buf, const f32x16* acc, int lane) {
#pragma unroll
  for (int b = 0; b < kN; ++b)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      f32x4 v = {acc[b][4 * q], acc[b][4 * q + 1], acc[b][4 * q + 2], acc[b][4 * q + 3]};
      *reinterpret_cast<f32x4*>(buf + ((b * 4 + q) * 64 + lane) * 4) = v;
    }
}
template <int kN>
__device__ __forceinline__ void acc_add_lds(f32x16* acc, const float* buf, float w, int lane) {
#pragma unroll
  for (int b = 0; b < kN; ++b)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(buf + ((b * 4 + q) * 64 + lane) * 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[b][4 * q + e] = fmaf(w, v[e], acc[b][4 * q + e]);
    }
}

// The lanes j (of 32, bits of the result) whose accumulators of either half hold a
// value that is not finite.  The kernels store these too and then write over them,
// in code marked as unlikely, so that the registers of the main loop are laid out
// without it (500 rows x 16,001 keys, 8 heads of 128 on 2, the step: 903 us without
// the check, 906 with it, 918 with a masked store and the branch not marked).
template <int kN>
__device__ __forceinline__ uint32_t not_finite(const f32x16* acc) {
  float t[4] = {0.f, 0.f, 0.f, 0.f};   // each 0, or NaN
#pragma unroll
  for (int b = 0; b < kN; ++b)
#pragma unroll
    for (int r = 0; r < 16; ++r) t[r & 3] = fmaf(acc[b][r], 0.f, t[r & 3]);
  const float x = (t[0] + t[1]) + (t[2] + t[3]);
  const uint64_t m = __ballot(x != x);
  return (uint32_t)m | (uint32_t)(m >> 32);
}

// Lane j's value, in every lane.
__device__ __forceinline__ int64_t of_lane(int64_t x, int j) {
  return (int64_t)(uint32_t)__builtin_amdgcn_readlane((int)x, j) |
         (int64_t)__builtin_amdgcn_readlane((int)(x >> 32), j) << 32;
}
// A uniform value that the compiler takes for a new one: what is computed from it
// again for the rare rows above is not kept in registers through the main loop.
__device__ __forceinline__ int opaque(int x) {
  asm volatile("" : "+s"(x));
  return x;
}

__device__ __forceinline__ int lane_id() {
  return (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
}

}  // namespace f32m
}  // namespace ls
