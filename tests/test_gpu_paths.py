"""Kernel variants that a rule on sizes chooses, at the sizes where each can go
wrong, against the fp64 oracle (needs an MI355X; bars as in the parity tests)."""
from __future__ import annotations

import pytest

from paper_2607_14952_amd import binding as B
from paper_2607_14952_amd import configs
from tests.test_gpu_parity import full_case

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu_ready():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.load_library()


def _f32(name, hq, hkv, d, dv, prefix, resp, page=64, shards=1, splits=2):
    return configs.C1.scaled(name=f"f32_{name}", n_q_heads=hq, n_kv_heads=hkv, head_dim=d,
                             head_dim_v=dv, prefix_len=prefix, resp_len=resp, page_size=page,
                             n_shards=shards, splits_per_shard=splits, table="perm")


@pytest.mark.parametrize("cfg", [
    # one row; one key more than a tile; head dimensions padded to 64, 96 and 128
    _f32("row", 4, 1, 64, 64, 33, 1),
    _f32("d40_dv72_g5", 5, 1, 40, 72, 515, 36, page=16),
    _f32("d124_dv8", 2, 2, 124, 8, 300, 34),
    # few rows, many key chunks whose partial sums are added (one short of whole)
    _f32("chunks", 2, 1, 64, 64, 9_001, 16),
    # enough 128-row groups that four row groups share the staged keys, whole
    # and with a ragged last one, over several key chunks
    _f32("shared_tiles", 8, 4, 96, 96, 4_103, 260),
    # response keys in several blocks and row chunks (five, the last ragged)
    _f32("dkdv_chunks", 8, 2, 128, 128, 100, 300),
    # the generic kernels: a width that is no multiple of 4, and one past 128
    _f32("generic_d66", 4, 2, 66, 64, 200, 33),
    _f32("generic_d160", 2, 1, 160, 160, 200, 33),
], ids=lambda c: c.name)
def test_f32_shapes(cfg):
    full_case(cfg)


def _bf16(name, prefix, resp, hq=16, hkv=2, page=256, shards=1, splits=2, **kw):
    # No planted keys: with all of them aimed at one row, dq is what is left of
    # large terms that cancel, and the bf16 rounding of out inside Delta alone
    # moves it by 9.2e-3 (10,017 keys, 100 planted, the rest in 64 bits; 8e-5
    # without planted keys).
    kw.setdefault("plant_frac", 0.0)
    return configs.C3.scaled(name=f"bf16_{name}", n_q_heads=hq, n_kv_heads=hkv, prefix_len=prefix,
                             resp_len=resp, page_size=page, n_shards=shards,
                             splits_per_shard=splits, **kw)


@pytest.mark.parametrize("cfg", [
    # dq over key chunks (few row tiles): one row, the last chunk one tile;
    # 16-position pages; two row tiles per KV head, the second ragged
    _bf16("dq_chunks_r1", 10_017, 1),
    _bf16("dq_chunks_p16", 5_003, 17, page=16),
    _bf16("dq_chunks_r20", 8_192, 20, shards=3),
    # enough row tiles that a few chunks only even out the last round
    _bf16("dq_rounds", 2_100, 1_120),
    # dk/dv row chunks of 128 rows up to 16 of them, the last one ragged
    _bf16("dkdv_r17", 300, 17),
    _bf16("dkdv_g4", 64, 519, hq=4, hkv=1),
], ids=lambda c: c.name)
def test_bf16_shapes(cfg):
    full_case(cfg)
