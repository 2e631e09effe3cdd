// Host rules of csrc/ls_internal.h for tests/test_plan_host.py.
#include "../include/longstraw.h"
#include "ls_internal.h"

extern "C" int64_t dkdv_launch_chunks(int n_q, int group, int n_kv_heads, int64_t n_keys) {
  return ls::dkdv_launch_chunks(n_q, group, n_kv_heads, n_keys);
}
extern "C" int64_t dkdv_part_keys(int n_q, int group, int n_kv_heads, int64_t n_resp) {
  return ls::dkdv_part_keys(n_q, group, n_kv_heads, n_resp);
}
// The bounds that the kernel of the launch beginning with split i0 sees; returns the
// launch's splits.
extern "C" int pack_splits(const ls_split* splits, int n, int i0, int64_t* begin, int64_t* end) {
  static ls::FwdArgs a;
  const int m = ls::pack_splits(a, splits + i0, n - i0);
  for (int i = 0; i < m; ++i) {
    begin[i] = a.split_begin(i);
    end[i] = a.split_end(i);
  }
  return m;
}
// Whether a launch of n splits of `keys` keys takes the fp32 forward's 128-row workgroups.
extern "C" int f32_fwd_wide(int n_q, int group, int n_kv_heads, int n, int keys) {
  static ls::FwdArgs a;
  a.n_q = n_q;
  a.group = group;
  a.n_kv_heads = n_kv_heads;
  a.n_splits = n;
  for (int i = 0; i < n; ++i) {
    a.split_lo[i] = i * keys;
    a.split_hi[i] = (i + 1) * keys;
  }
  return ls::f32_fwd_wide(a);
}
