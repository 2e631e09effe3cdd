"""The launch plan of a replay step on the CPU: the pieces of the forward cover
each shard's keys once, and a cyclic step's table names every owned page in
its shard's range, with the partly filled last page and the response in place."""
import numpy as np
import pytest

from paper_2607_14952_amd import configs
from paper_2607_14952_amd.replay import cyclic_shards, fine_splits

BASE = configs.C3


@pytest.mark.parametrize("kw", [
    dict(prefix_len=131_075, resp_len=1, splits_per_shard=8), dict(prefix_len=1, resp_len=1),
    dict(prefix_len=1000, resp_len=7, page_size=16), dict(prefix_len=0, resp_len=5, n_shards=1),
    dict(), dict(prefix_len=5000, resp_len=129, dtype="f32", head_dim=64, head_dim_v=64),
], ids=str)
def test_pieces_cover_each_split(kw):
    cfg = BASE.scaled(**kw)
    splits = [[r for r in cfg.splits() if r[0] < r[1] and b <= r[0] and r[1] <= e]
              for b, e in cfg.shard_ranges() if b < e]
    fine = fine_splits(cfg, splits)
    assert fine[-1] == splits[-1]
    for whole, parts in zip(splits, fine):
        assert parts[0][0] == whole[0][0] and parts[-1][1] == whole[-1][1]
        assert all(b < e for b, e in parts)
        assert all(x[1] == y[0] for x, y in zip(parts, parts[1:]))
        assert {r[0] for r in whole} <= {r[0] for r in parts}   # no piece spans two splits
    assert sum(map(len, fine)) <= max(1025, sum(map(len, splits)))


def test_headline_step_stays_whole():
    splits = [[r for r in BASE.splits() if b <= r[0] and r[1] <= e]
              for b, e in BASE.shard_ranges()]
    assert fine_splits(BASE, splits) == splits


@pytest.mark.parametrize("prefix,page,shards", [(256 * 61 + 100, 256, 8), (256 * 64, 256, 8),
                                                (100_003, 64, 8), (50, 64, 8), (16 * 13 + 1, 16, 3),
                                                (16 * 5, 16, 8)])
def test_cyclic_table(prefix, page, shards):
    cfg = BASE.scaled(prefix_len=prefix, page_size=page, n_shards=shards, resp_len=page + 3,
                      ownership="cyclic")
    ranges, order = cyclic_shards(cfg)
    assert sorted(order) == list(range(cfg.n_prefix_pages))
    assert ranges[-1] == (prefix, cfg.kv_len)
    owners = [c for c in range(shards) if cfg.shard_len(c)]
    seen = np.zeros(prefix, dtype=int)
    for c, (b, e) in zip(owners, ranges):
        assert 0 <= b < e <= prefix and b % page == 0
        v = np.arange(b, e)
        logical = np.asarray(order)[v // page] * page + v % page
        assert np.all(logical // page % shards == c)
        seen[logical] += 1
    assert np.all(seen == 1)
    if prefix % page:   # the response goes on in the same physical page
        assert order[-1] == cfg.n_prefix_pages - 1


@pytest.mark.parametrize("kw", [dict(prefix_len=256 * 61 + 100), dict(prefix_len=64 * 37 + 1, page_size=64),
                                dict(prefix_len=16 * 61 + 5, page_size=16),
                                dict(prefix_len=256 * 3)], ids=str)
def test_cyclic_step_names_each_shards_own_store(kw):
    """A cyclic step's shards, shard_splits and splits are ranges of the shards' own
    stores, whose tables begin with the owned pages, whatever store the step itself
    reads them through."""
    import torch

    from paper_2607_14952_amd.replay import ReplayStep
    cfg = BASE.scaled(resp_len=21, splits_per_shard=2, ownership="cyclic", **kw)
    n_pages = cfg.n_logical_pages
    table = np.random.default_rng(1).permutation(n_pages).astype(np.int32)
    pool = torch.zeros((n_pages, 1, 1, 1), dtype=torch.bfloat16)
    step = ReplayStep(cfg, dict(q=torch.zeros((21, 16, 256), dtype=torch.bfloat16), k_pool=pool,
                                v_pool=pool, page_table=torch.from_numpy(table)), backward=False)
    assert step.cyclic
    owners = [c for c in range(cfg.n_shards) if cfg.shard_len(c)]
    assert step.shards == [(0, cfg.shard_len(c)) for c in owners] + [(cfg.prefix_len, cfg.kv_len)]
    assert len(step.shard_kv) == len(step.shards) and step.shard_kv[-1] is step.kv
    for s, c in enumerate(owners):
        pages = cfg.shard_pages(c)
        assert np.array_equal(step.shard_kv[s].page_table.numpy()[:len(pages)], table[pages])
    for (b, e), parts, (i, j) in zip(step.shards, step.shard_splits, step.groups):
        assert parts == step.splits[i:j]
        assert parts[0][0] == b and parts[-1][1] == e
        assert all(x[1] == y[0] for x, y in zip(parts, parts[1:]))
    assert sorted(x for g in step.groups for x in range(*g)) == list(range(len(step.splits)))


def test_merge_groups_rejects():
    import ctypes

    from paper_2607_14952_amd import binding as B
    from tests.test_abi import FAKE
    lib = B.load_library()

    def call(groups, n_parts=8, dv=256, dtype=B.LS_BF16, flags=0, out=FAKE * 300, gout=FAKE * 200):
        k = len(groups)
        b = (ctypes.c_int32 * max(k, 1))(*[g[0] for g in groups])
        e = (ctypes.c_int32 * max(k, 1))(*[g[1] for g in groups])
        return lib.ls_lse_merge_groups(FAKE, FAKE * 100, n_parts, b, e, k, 16, 16, dv, dtype, gout,
                                       FAKE * 250, out, FAKE * 400, flags, None)

    assert call([]) == -1
    assert call([(0, 0)]) == -1
    assert call([(0, 4), (4, 9)]) == -1
    assert call([(-1, 4)]) == -1
    assert call([(0, 8)] * 65) == -2
    assert call([(0, 4), (4, 8)], dv=254) == -2
    assert call([(0, 4), (4, 8)], dtype=7) == -2
    assert call([(0, 4), (4, 8)], flags=2) == -2
    assert call([(0, 4), (4, 8)], out=FAKE + 64) == -4
    assert call([(0, 4), (4, 8)], gout=FAKE + 4) == -1
