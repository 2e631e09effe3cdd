"""The top-k kernel's own source on the CPU (topk_host.cpp): the selection with each
wave ahead of the others in turn, as far as the barriers let it."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2607_14952_amd", "csrc")
pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="g++ missing")


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("topk_host")
    with open(os.path.join(CSRC, "dsa_select.hip")) as f:
        src = f.read()
    kernel = src[src.index("// ---------------------------------------------------------------- top-k"):]
    launch = kernel[kernel.index("// Keys of each of a row's chunks"):kernel.rindex("}  // namespace ls")]
    (tmp / "topk_section.inc").write_text(kernel[:kernel.index("}  // namespace")])
    (tmp / "topk_launch.inc").write_text(launch)
    so = tmp / "topk_host.so"
    cmd = ["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-Wno-unknown-pragmas", "-I",
           os.path.join(HERE, "host_shim"), "-I", CSRC, "-I", str(tmp),
           os.path.join(HERE, "topk_host.cpp"), "-o", str(so)]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout[-4000:]
    return ctypes.CDLL(str(so))


def order_key(x):
    """The library's order of scores, as integers: -0 below +0."""
    key = x.view(np.int32)
    return np.where(key < 0, key ^ 0x7FFFFFFF, key).astype(np.int64)


def check(lib, x, k, n_chunks=1, orders=(0, 1, 2)):
    """The kernel's selection from the rows of x, against a stable sort's."""
    rows, n = x.shape
    flat = np.zeros(rows * n + 4, np.float32)
    at = -flat.ctypes.data // 4 % 4     # 16-byte aligned
    buf = flat[at:at + rows * n].reshape(rows, n)
    buf[:] = x
    c = ctypes
    for order in orders:
        pos, sc = np.full((rows, k), -7, np.int32), np.zeros((rows, k), np.float32)
        parted = lib.topk_host(c.c_void_p(buf.ctypes.data), c.c_int64(n), None, rows, c.c_int64(n),
                               c.c_int64(5), k, c.c_void_p(pos.ctypes.data),
                               c.c_void_p(sc.ctypes.data), c.c_int64(k), n_chunks, order)
        assert not parted, f"threads wait at different barriers (order {order})"
        for r in range(rows):
            want = np.sort(np.argsort(-order_key(x[r]), kind="stable")[:k])
            assert np.array_equal(pos[r], want + 5), f"order {order}"
            assert np.array_equal(sc[r].view(np.int32), x[r, want].view(np.int32))


@pytest.mark.parametrize("value,n,k", [(-2.5, 5_000, 300), (-3.0e38, 4_500, 2_000), (1.5, 5_000, 9)])
def test_many_keys_in_the_threshold_bin(lib, value, n, k):
    """More keys share the threshold's first digit than the LDS list holds: the row is
    passed over again.  At -2 and below, that digit's own count lies where the next
    histogram begins, which no wave may clear before every wave has read it."""
    x = np.full((1, n), value, np.float32)
    check(lib, x, k)
    x[0, ::7] *= np.float32(1 + 2.0 ** -20)   # two keys in one bin
    check(lib, x, k)


@pytest.mark.parametrize("kind", ["normal", "ties", "mostly_inf"])
@pytest.mark.parametrize("n,k,n_chunks", [(3_001, 300, 1), (66_000, 700, 1), (140_001, 512, 2)])
def test_selection(lib, kind, n, k, n_chunks):
    rng = np.random.default_rng(n + k)
    x = rng.standard_normal((1, n)).astype(np.float32)
    if kind == "ties":
        x = np.round(x * 4) / np.float32(4)
    elif kind == "mostly_inf":
        x[:, k // 2:] = -np.inf
    check(lib, x, k, n_chunks, orders=(0, 1) if n < 10_000 else (1,))


def test_nan_does_not_fill_up_a_bound_too_high(lib):
    """The sampled blocks hold all the large keys, so that fewer than k of the row's keys
    reach the bound; NaNs with the sign bit set (the lowest of the key order) pass the
    bound's float comparison and bring the candidates to k or more.  The row's selection
    is of its finite keys all the same."""
    n, k = 66_000, 700
    rng = np.random.default_rng(3)
    x = rng.uniform(-1, 1, (1, n)).astype(np.float32)
    sampled = np.concatenate([np.arange(32) + (j * (n // 512) & ~31) for j in range(512)])
    x[0, rng.choice(sampled, 450, replace=False)] = rng.uniform(5, 9, 450).astype(np.float32)
    others = np.setdiff1d(np.arange(n), sampled)
    x.view(np.uint32)[0, rng.choice(others, 600, replace=False)] = 0xFFC00000
    check(lib, x, k)


def test_chunks_keep_the_sampled_path(lib):
    """Every chunk that the rule cuts, the last one too, has the 65,536 keys from which
    on a row is sampled; the launch's chunks are the rule's."""
    c = ctypes
    cut = 0
    for n in [1_029_369, *range(131_072, 1_048_577, 1_073)]:
        for rows, k in ((1, 2048), (3, 700), (40, 64)):
            m = lib.topk_chunk_count(c.c_int64(rows), c.c_int64(n), k)
            assert 1 <= m <= 16
            if m > 1:
                seg = lib.topk_chunk_len(c.c_int64(n), m)
                assert seg % 256 == 0 and (m - 1) * seg + 65_536 <= n <= m * seg, (n, m)
                cut += 1
    assert cut > 100


@pytest.mark.parametrize("width", [64, 256])
def test_smooth_rows_stay_on_the_sampled_path(lib, width):
    """Neighbouring scores of an index resemble each other.  Rows smoothed over so many
    positions select as those in random order do, without the passes over the whole
    row that follow a bound too high (told by the barriers passed)."""
    n, k = 65_536, 2_048
    window = np.zeros(n)
    window[:width] = np.hanning(width + 2)[1:-1]

    def barriers(x):
        check(lib, x[None], k, orders=(0,))
        return lib.topk_barriers()
    rows = [np.random.default_rng(s).standard_normal(n) for s in range(24)]
    usual = barriers(rows[0].astype(np.float32))
    smooth = [np.fft.irfft(np.fft.rfft(r) * np.fft.rfft(window), n).astype(np.float32) for r in rows]
    assert sum(barriers(r / r.std()) != usual for r in smooth) == 0
