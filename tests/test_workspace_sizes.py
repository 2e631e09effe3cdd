"""Workspace sizes on the CPU: one made for some rows serves any call with fewer
rows or a smaller q_pos0, as blockwise replay's ragged last block relies on."""
import ctypes
import os

import pytest

from paper_2607_14952_amd import binding as B
from tests.test_abi import good_params

pytestmark = pytest.mark.skipif(not os.path.exists(B.LIB_PATH),
                                reason="liblongstraw.so not built (run __graft_entry__.build())")


@pytest.mark.parametrize("kw", [dict(), dict(n_q_heads=4, n_kv_heads=4),
                                dict(dtype=B.LS_F32, head_dim=96, head_dim_v=64, n_q_heads=6),
                                dict(dtype=B.LS_F32, head_dim=160, head_dim_v=160)],
                         ids=["bf16", "bf16_g1", "f32", "f32_generic"])
def test_backward_workspace_grows_with_rows(kw):
    def size(n_q, q_off):
        p = good_params(n_q=n_q, q_pos0=4096 + q_off, n_logical_pages=1 << 16, **kw)
        return B.load_library().ls_prefix_attn_bwd_workspace_size(ctypes.byref(p))

    rows = [1, 2, 7, 15, 16, 17, 31, 33, 64, 127, 128, 129, 250, 257, 511, 600, 1111, 2047, 2048,
            2049, 4096, 5000, 8192]
    for off in (0, 100, 4096):
        sizes = [size(n, off) for n in rows]
        assert sizes == sorted(sizes)
        assert all(size(n, off) <= size(n, off + 77) for n in rows)
