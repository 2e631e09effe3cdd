// The top-k kernel of csrc/dsa_select.hip on the CPU: each thread of a workgroup
// is a fiber, wave operations meet their 64 lanes, and between two barriers one
// wave after another runs as far as it can, in a given order.  So a wave that
// may get ahead of the others between barriers does, every time, and threads
// that wait at different barriers are reported instead of hanging.  (Lanes of a
// wave run one after another between its wave operations, which asks more of
// the code than lockstep does.)
#include <math.h>
#include <stdio.h>
#include <string.h>
#include <ucontext.h>

#include <algorithm>
#include <memory>
#include <vector>

#include "ls_internal.h"

namespace emu {
constexpr int kMax = 512, kStack = 128 << 10;
enum State { kRun, kWave, kBarrier, kDone };
struct Thread {
  ucontext_t ctx;
  State state;
  int site;        // line of the operation it waits at
  uint64_t in;     // its value in a wave operation
};
struct Group {
  std::unique_ptr<Thread[]> t{new Thread[kMax]};
  std::vector<char> stacks = std::vector<char>((size_t)kMax * kStack);
  ucontext_t main;
  int n = 0, cur = 0;
  dim3 block;
  void (*body)(const ls::TopkArgs&) = nullptr;
  const ls::TopkArgs* args = nullptr;
  bool diverged = false;
  int barriers = 0;
};
Group g;
int order = 0;           // 0: waves ascending, 1: descending, 2: odd waves first
uint64_t values[64];     // of the wave operation just met, by lane
struct Index { unsigned x, y, z; };
inline Index thread() { return {(unsigned)g.cur, 0, 0}; }
inline Index block() { return {g.block.x, g.block.y, g.block.z}; }
inline int lane() { return g.cur & 63; }
inline const uint64_t* wait(State s, int site, uint64_t in) {
  Thread& t = g.t[g.cur];
  t.state = s;
  t.site = site;
  t.in = in;
  swapcontext(&t.ctx, &g.main);
  return values;
}
void entry() {
  g.body(*g.args);
  g.t[g.cur].state = kDone;
  swapcontext(&g.t[g.cur].ctx, &g.main);
}
// Lanes of wave w until all wait at a barrier or are done; false when they part.
bool run_wave(int w) {
  Thread* t = &g.t[64 * w];
  for (;;) {
    for (int l = 0; l < 64; ++l)
      if (t[l].state == kRun) {
        g.cur = 64 * w + l;
        swapcontext(&g.main, &t[l].ctx);
      }
    for (int l = 1; l < 64; ++l)
      if (t[l].state != t[0].state || t[l].site != t[0].site) return false;
    if (t[0].state != kWave) return true;
    for (int l = 0; l < 64; ++l) {
      values[l] = t[l].in;
      t[l].state = kRun;
    }
  }
}
}  // namespace emu

// A wave operation leaves all lanes' values to each lane, which picks its result.
#define EMU_WAVE(value) emu::wait(emu::kWave, __LINE__, (uint64_t)(value))
inline uint64_t emu_ballot(const uint64_t* v) {
  uint64_t m = 0;
  for (int l = 0; l < 64; ++l) m |= (uint64_t)(v[l] != 0) << l;
  return m;
}
inline uint32_t emu_sum(const uint64_t* v) {
  uint32_t s = 0;
  for (int l = 0; l < 64; ++l) s += (uint32_t)v[l];
  return s;
}
inline uint32_t emu_lane(const uint64_t* v, int l) { return (uint32_t)v[l < 64 ? l : emu::lane()]; }
inline uint32_t emu_mbcnt(uint32_t m, uint32_t x, int first) {
  const int below = emu::lane() - first;
  return x + (below <= 0 ? 0 : __builtin_popcountll(m & ((uint64_t(1) << std::min(below, 32)) - 1)));
}
template <typename T> inline T min(T a, T b) { return a < b ? a : b; }
template <typename T> inline T max(T a, T b) { return a > b ? a : b; }
template <typename T> inline T atomicAdd(T* p, T v) { const T o = *p; *p += v; return o; }
inline float as_float(uint32_t u) { float f; memcpy(&f, &u, 4); return f; }
inline uint32_t as_uint(float f) { uint32_t u; memcpy(&u, &f, 4); return u; }
#define __shared__ static
#define __syncthreads() emu::wait(emu::kBarrier, __LINE__, 0)
#define __ballot(p) emu_ballot(EMU_WAVE(p))
#define __reduce_add_sync(mask, v) emu_sum(EMU_WAVE(v))
#define __shfl(v, l) emu_lane(EMU_WAVE(v), l)
#define __shfl_down(v, d) emu_lane(EMU_WAVE(v), emu::lane() + (d))
#define __popcll __builtin_popcountll
#define __builtin_amdgcn_mbcnt_lo(m, x) emu_mbcnt(m, x, 0)
#define __builtin_amdgcn_mbcnt_hi(m, x) emu_mbcnt(m, x, 32)
#define __float_as_uint as_uint
#define __uint_as_float as_float
#define threadIdx emu::thread()
#define blockIdx emu::block()
#define hipLaunchKernelGGL(kernel, grid, block, lds, stream, args) \
  emu_launch(kernel, grid, block, args)
static void emu_launch(void (*kernel)(ls::TopkArgs), dim3 grid, dim3 block, const ls::TopkArgs& a);

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
namespace ls {
namespace {
#include "topk_section.inc"    // the kernel, cut out of dsa_select.hip
}  // namespace
#include "topk_launch.inc"     // topk_chunks and launch_topk
}  // namespace ls

#undef threadIdx
#undef blockIdx
static void emu_launch(void (*)(ls::TopkArgs), dim3 grid, dim3 block, const ls::TopkArgs& a) {
  using namespace emu;
  g.n = (int)block.x;
  g.args = &a;
  g.body = [](const ls::TopkArgs& x) { ls::topk_kernel(x); };
  const int waves = g.n / 64;
  for (unsigned y = 0; y < grid.y; ++y)
    for (unsigned x = 0; x < grid.x && !g.diverged; ++x) {
      g.block = dim3(x, y);
      for (int i = 0; i < g.n; ++i) {
        Thread& t = g.t[i];
        getcontext(&t.ctx);
        t.ctx.uc_stack.ss_sp = g.stacks.data() + (size_t)i * kStack;
        t.ctx.uc_stack.ss_size = kStack;
        t.ctx.uc_link = nullptr;
        makecontext(&t.ctx, entry, 0);
        t.state = kRun;
        t.site = 0;
      }
      for (bool done = false; !done;) {
        for (int i = 0; i < waves; ++i) {
          const int w = order == 0 ? i : order == 1 ? waves - 1 - i : (2 * i + 1) % (waves + 1);
          if (!run_wave(w)) g.diverged = true;
        }
        for (int i = 1; i < g.n; ++i)
          if (g.t[i].state != g.t[0].state || g.t[i].site != g.t[0].site) g.diverged = true;
        if (g.diverged) {
          for (int i = 0; i < g.n; ++i)
            if (i % 64 == 0 || g.t[i].site != g.t[i - 1].site)
              fprintf(stderr, "from thread %d on: state %d at line %d\n", i, g.t[i].state, g.t[i].site);
          return;
        }
        done = g.t[0].state == kDone;
        g.barriers += !done;
        for (int i = 0; i < g.n && !done; ++i) g.t[i].state = kRun;
      }
    }
}

extern "C" int topk_chunk_count(int64_t n_rows, int64_t n, int k) {
  return ls::topk_chunks(n_rows, n, k);
}

// Barriers that the workgroups of the last call passed.
extern "C" int topk_barriers() { return emu::g.barriers; }

extern "C" int topk_chunk_len(int64_t n, int n_chunks) {
  return (int)ls::topk_chunk_len(n, n_chunks);
}

// ls_topk_select_ws on host memory; n_chunks 0: as topk_chunks says.  Nonzero
// when the waves of a workgroup waited at different barriers.
extern "C" int topk_host(const float* scores, int64_t ld, const int32_t* positions, int32_t n_rows,
                         int64_t n, int64_t pos_offset, int32_t k, int32_t* out_pos,
                         float* out_scores, int64_t out_ld, int32_t n_chunks, int32_t order) {
  ls::TopkArgs a{};
  a.scores = scores;
  a.positions = positions;
  a.out_pos = out_pos;
  a.out_scores = out_scores;
  a.ld = ld;
  a.out_ld = out_ld;
  a.n = n;
  a.pos_offset = pos_offset;
  a.n_rows = n_rows;
  a.k = k;
  emu::order = order;
  emu::g.diverged = false;
  emu::g.barriers = 0;
  if (n_chunks == 0) n_chunks = ls::topk_chunks(n_rows, n, k);
  std::vector<int32_t> cand((size_t)n_rows * n_chunks * k);
  std::vector<float> cand_scores(cand.size());
  ls::launch_topk(a, n_chunks, cand.data(), cand_scores.data(), nullptr);
  return emu::g.diverged ? 1 : 0;
}
