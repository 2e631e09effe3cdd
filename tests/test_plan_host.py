"""Launch plans that the host code makes (csrc/ls_internal.h), on the CPU."""
import ctypes
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2607_14952_amd", "csrc")
pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="g++ missing")
I64 = ctypes.c_int64


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    so = tmp_path_factory.mktemp("plan_host") / "plan_host.so"
    cmd = ["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", os.path.join(HERE, "host_shim"),
           "-I", CSRC, os.path.join(HERE, "plan_host.cpp"), "-o", str(so)]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout[-4000:]
    lib = ctypes.CDLL(str(so))
    lib.dkdv_launch_chunks.restype = lib.dkdv_part_keys.restype = I64
    return lib


ROWS = [1, 15, 16, 17, 33, 64, 77, 128, 250, 1_111, 2_048, 2_049, 4_096, 5_000]


@pytest.mark.parametrize("group,hkv", [(8, 2), (1, 4), (32, 1), (16, 2)])
def test_dkdv_partials_fit_what_is_reserved(lib, group, hkv):
    """Whatever keys of the response a launch takes, its chunks' partial sums fit, and
    what is reserved is no more than the largest launch's twice over (or one round of
    workgroups' more)."""
    last = {}
    for n_q in ROWS:
        for n_resp in sorted({n_q, n_q + 77, n_q + 4_096, 8_192 + n_q}):
            room = lib.dkdv_part_keys(n_q, group, hkv, I64(n_resp))
            used = [lib.dkdv_launch_chunks(n_q, group, hkv, I64(n)) * n
                    for n in {*range(1, min(n_resp, 700) + 1), *range(1, n_resp + 1, 61), n_resp}]
            assert max(used) <= room <= 2 * max(used) + 512 * 128 // hkv, (n_q, n_resp)
            assert room >= lib.dkdv_part_keys(n_q, group, hkv, I64(n_resp - 1))
            assert room >= last.get(n_resp - n_q, 0)
            last[n_resp - n_q] = room


def test_block_of_2048_reserves_the_chunks_it_takes(lib):
    """2,048 tokens of 16 heads on 2, the last block of an 8,192-token response: eight
    chunks, where sixteen would be the most for fewer keys."""
    assert lib.dkdv_launch_chunks(2_048, 8, 2, I64(8_192)) == 8
    assert lib.dkdv_part_keys(2_048, 8, 2, I64(8_192)) == 8 * 8_192


BIG = 1 << 32


@pytest.mark.parametrize("splits", [
    [(0, 1)], [(7 * i, 7 * i + 5) for i in range(1_000)],
    # one that no 32-bit offset reaches, first, last and between others
    [(5, BIG + 5)], [(3, 9), (9, 2 * BIG), (2 * BIG, 2 * BIG + 1)],
    # ends at and one past the offsets' reach from the launch's first key
    [(11, 20), (20, 11 + BIG - 1)], [(11, 20), (20, 11 + BIG)],
    [(i << 30, (i + 1) << 30) for i in range(1, 40)],
], ids=["one", "many", "long", "long_between", "reach", "past", "gibi"])
def test_split_bounds_survive_packing(lib, splits):
    arr = (I64 * (2 * len(splits)))(*[x for s in splits for x in s])
    begin, end = (I64 * 448)(), (I64 * 448)()
    got, i = [], 0
    while i < len(splits):
        m = lib.pack_splits(arr, len(splits), i, begin, end)
        assert 1 <= m <= 448 and i + m <= len(splits)
        got += list(zip(begin[:m], end[:m]))
        i += m
    assert got == splits


@pytest.mark.parametrize("n_q,hkv,splits,keys,wide", [
    # rows of 32 heads on 4 (8 on 2): few workgroups, one round or two of them, more
    (64, 1, 3, 256, 0), (48, 4, 8, 64, 1), (48, 4, 8, 256, 0), (91, 4, 5, 64, 1),
    (91, 4, 5, 1_024, 0), (91, 4, 9, 64, 1), (91, 4, 9, 256, 1), (91, 4, 9, 4_096, 1),
    (91, 4, 20, 256, 1),
])
def test_f32_forward_workgroups(lib, n_q, hkv, splits, keys, wide):
    """The measured better of the two workgroup sizes."""
    assert lib.f32_fwd_wide(n_q, 8, hkv, splits, keys) == wide
