// Host rules of csrc/ls_internal.h for tests/test_plan_host.py.
#include "ls_internal.h"

extern "C" int64_t dkdv_launch_chunks(int n_q, int group, int n_kv_heads, int64_t n_keys) {
  return ls::dkdv_launch_chunks(n_q, group, n_kv_heads, n_keys);
}
extern "C" int64_t dkdv_part_keys(int n_q, int group, int n_kv_heads, int64_t n_resp) {
  return ls::dkdv_part_keys(n_q, group, n_kv_heads, n_resp);
}
