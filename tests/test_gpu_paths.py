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
    # a response of a few keys, whose backward runs on the generic kernels
    _f32("few_keys", 8, 4, 128, 128, 300, 6),
    # short splits: 128-row workgroups though they are fewer than the CUs
    _f32("short_splits", 32, 4, 64, 64, 1_000, 91, splits=10),
    # dk/dv of few rows on the generic kernel, dq on the matrix cores; the reverse
    _f32("few_rows", 2, 1, 64, 64, 300, 10),
    _f32("few_dq_keys", 32, 2, 128, 128, 300, 4),
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


@pytest.mark.parametrize("flag", [0, B.FLAG_BF16_NUMERATOR], ids=["f32num", "bf16num"])
@pytest.mark.parametrize("R,H,Dv,groups", [
    # the narrow kernel (16 waves share an item's parts): one row; units of more
    # than 8 parts; groups of one part and of many, out of order; items that do
    # not fill a workgroup
    (1, 2, 64, [(0, 3), (3, 4)]),
    (2, 3, 20, [(200, 201), (0, 200), (201, 209)]),
    (16, 16, 256, [(32 * i, 32 * i + 32) for i in range(8)] + [(256, 257)]),
    # the most groups; one group; past the narrow kernel's largest call
    (3, 4, 32, [(i, i + 1) for i in range(64)]),
    (5, 4, 64, [(0, 21)]),
    (520, 1, 256, [(0, 5), (5, 14)]),
], ids=["row", "ragged", "r16", "g64", "one_group", "wide"])
def test_merge_groups(R, H, Dv, groups, flag):
    """Both levels in one launch against the oracle's merge of each group and of
    the groups' results (for the bf16 numerator, its bf16 composition of them and the
    library's own in two steps); rows and groups with no key at all included."""
    import numpy as np
    import torch

    import oracle as O
    from paper_2607_14952_amd import inputs
    from tests._gpu import host, lse_err, rel_l2
    n = max(e for _, e in groups)
    o, lse = inputs.merge_parts(77 + n, n, R, H, Dv)
    b0, e0 = groups[0]
    lse[b0:e0, 0, 0] = -np.inf          # a whole group empty for one row
    o[b0:e0, 0, 0] = 0.0
    f32 = dict(dtype=torch.float32, device="cuda")
    go, gl = torch.full((len(groups), R, H, Dv), 7.0, **f32), torch.full((len(groups), H, R), 7.0, **f32)
    out, l = torch.empty((R, H, Dv), **f32), torch.empty((H, R), **f32)
    B.lse_merge_groups(torch.from_numpy(o).cuda(), torch.from_numpy(lse).cuda(), groups,
                       group_out=go, group_lse=gl, out=out, lse=l, flags=flag)
    torch.cuda.synchronize()
    parts = [O.lse_merge(list(o[b:e]), list(lse[b:e])) for b, e in groups]
    for k, (ro, rl) in enumerate(parts):
        assert rel_l2(host(go[k]), ro) <= 1e-6 and lse_err(host(gl[k]), rl) <= 1e-5
    want, want_l = O.lse_merge([p[0] for p in parts], [p[1] for p in parts])
    assert lse_err(host(l), want_l) <= 1e-5
    if not flag:
        assert rel_l2(host(out), want) <= 1e-6
        return
    # bf16 numerator: the two-step composition's values.  The narrow kernel's weights
    # may differ in the last fp32 bits, which now and then rounds a term or a running
    # sum to the other neighbour: an ulp, 2^-7 of no more than the sum of the terms'
    # magnitudes, and no element meets it more than twice here.
    two, _ = B.lse_merge(go, gl, out_dtype=torch.float32, flags=flag)
    with np.errstate(invalid="ignore"):                    # [groups, H, R]
        w = np.where(np.isfinite(host(l)), np.exp(host(gl) - host(l)), 0.0)
    mag = (w.transpose(0, 2, 1)[..., None] * np.abs(host(go))).sum(0)
    diff = np.abs(host(two) - host(out))
    assert (diff <= 1e-6 * (np.abs(host(two)) + 1e-30)).mean() >= 0.99
    assert np.all(diff <= 2 * 2.0 ** -7 * mag + 1e-30)
    ref, _ = O.lse_merge_bf16_numerator(list(host(go)), list(host(gl)))
    assert rel_l2(host(out), ref) <= 2.0 ** -8


@pytest.mark.parametrize("R,topk,heads", [(1, 2048, 128), (3, 515, 128), (9, 300, 256),
                                          (24, 2048, 128), (130, 700, 128)])
def test_sparse_key_chunks(R, topk, heads):
    """Few tokens: each one's key list is cut into chunks whose results are
    merged (the forward) or added (dq), among them tokens whose selection is
    mostly pads, with fewer tiles than chunks.  The lists straddle the batches
    in which they are resolved.  A workspace too small for the partial results
    (the size before any chunk) gives the same within rounding, and
    accumulation adds to dq once."""
    import ctypes

    import numpy as np
    import torch

    from paper_2607_14952_amd import inputs
    from paper_2607_14952_amd.replay import to_device
    from tests._gpu import announce, host, rel_l2
    from tests.test_gpu_sparse import run
    cfg = configs.C5.scaled(name=f"sparse_chunks_{R}", prefix_len=8192, resp_len=R, topk=topk,
                            n_q_heads=heads)
    h = inputs.sparse_inputs(cfg)
    idx = h["idx"].copy()
    if R > 2:
        idx[1, 3:] = -1            # one tile, where the others have many
        idx[2, : topk // 2] = -1
    h = dict(h, idx=idx)
    run(cfg, h)
    q, lat, di = to_device(h["q"]), to_device(h["latent_pool"]), to_device(idx)
    kv = B.PagedKV(lat, lat, to_device(h["page_table"]))
    kw = dict(prefix_len=cfg.prefix_len, q_pos0=cfg.q_pos0, scale=cfg.scale)
    do = to_device(h["d_out"])
    out, lse = B.sparse_attn_fwd(q, kv, di, **kw)
    dq = B.sparse_attn_bwd(q, kv, di, do, out, lse, **kw)
    pad = lambda n: (n + 255) // 256 * 256  # noqa: E731
    lists = pad(R * -(-(topk + R) // 32) * 32 * 4) + pad(R * 4)
    small = torch.empty(lists + 2 * pad(R * heads * 4), dtype=torch.uint8, device="cuda")
    announce(f"sparse R={R}: workspace without partial results")
    out1, _ = B.sparse_attn_fwd(q, kv, di, workspace=small[:lists], **kw)
    acc = torch.ones_like(dq)
    B.sparse_attn_bwd(q, kv, di, do, out, lse, dq=acc, workspace=small,
                      flags=B.FLAG_ACCUMULATE_DQ, **kw)
    acc2 = torch.ones_like(dq)
    B.sparse_attn_bwd(q, kv, di, do, out, lse, dq=acc2, flags=B.FLAG_ACCUMULATE_DQ, **kw)
    torch.cuda.synchronize()
    # P and dS are rounded to bf16 relative to another maximum: 2^-9 each
    assert rel_l2(host(out1), host(out)) <= 2.0 ** -8
    assert rel_l2(host(acc) - 1, host(dq)) <= 2.0 ** -8
    assert rel_l2(host(acc2) - 1, host(dq)) <= 1e-5
    p = B._sparse_params(q, kv, **kw)
    assert lists <= B.load_library().ls_sparse_attn_workspace_size(ctypes.byref(p), topk, 0) <= 64 << 20


@pytest.mark.parametrize("kind", ["normal", "ties", "equal", "mostly_inf", "ascending"])
@pytest.mark.parametrize("rows,n,k,ld_pad", [
    (3, 300_003, 2048, 1),      # several chunks a row, a ragged last one
    (1, 1_050_000, 1, 0),       # the most chunks
    (2, 262_145, 700, 3),       # rows that are not 16-byte aligned
    (40, 200_000, 64, 0), (5, 70_001, 2048, 3), (2, 5_000, 300, 0),
], ids=["r3", "r1", "unaligned", "r40", "whole", "short"])
def test_topk_shared_rows(rows, n, k, ld_pad, kind):
    """The selection equals a stable sort's (ties to the lower position) however
    a row is shared, with given positions too."""
    import numpy as np
    import torch
    rng = np.random.default_rng(rows * 1000 + k)
    x = rng.standard_normal((rows, n + ld_pad)).astype(np.float32)
    if kind == "ties":
        x = np.round(x * 4) / 4 * np.float32(1.0)
        x[x == 0] = np.where(rng.random((x == 0).sum()) < 0.5, 0.0, -0.0)
    elif kind == "equal":
        x[:] = -2.5
    elif kind == "mostly_inf":
        x[:, k // 2:] = -np.inf
    elif kind == "ascending":    # the largest keys all in the last chunk
        x.sort(axis=1)
    sc = torch.from_numpy(x).cuda()
    pos = np.sort(rng.choice(1 << 30, size=n + ld_pad, replace=False)).astype(np.int32)
    pos = np.broadcast_to(pos, x.shape).copy()
    print(f"[gpu] top-k {kind} rows={rows} n={n} k={k}", flush=True)
    idx, val = B.topk_select(sc, k, n=n, pos_offset=7)
    named, _ = B.topk_select(sc, k, n=n, positions=torch.from_numpy(pos).cuda())
    torch.cuda.synchronize()
    # the key order of the library: -0 below +0
    key = x[:, :n].view(np.int32)
    key = np.where(key < 0, key ^ 0x7FFFFFFF, key)
    for r in range(rows):
        want = np.sort(np.argsort(-key[r].astype(np.int64), kind="stable")[:k])
        assert np.array_equal(idx[r].cpu().numpy(), want + 7)
        assert np.array_equal(val[r].cpu().numpy().view(np.int32), x[r, want].view(np.int32))
        assert np.array_equal(named[r].cpu().numpy(), pos[r, want])


@pytest.mark.parametrize("R,P,heads", [(1, 1_000, 8), (33, 4_100, 16), (70, 16_385 + 32, 24),
                                       (40, 33_000, 32)])
def test_dsa_scores_chunks(R, P, heads):
    """Key chunks of a few tiles (the last one short) against fp64 products."""
    import numpy as np
    import torch

    from paper_2607_14952_amd import inputs
    from paper_2607_14952_amd.replay import to_device
    from tests._gpu import host, rel_l2
    h = inputs.dsa_index_inputs(5, R, heads, P, 64)
    d = {k: to_device(v) for k, v in h.items()}
    print(f"[gpu] dsa scores R={R} P={P}", flush=True)
    s = B.dsa_index_scores(d["q_index"], d["w_index"], d["k_index_pool"], d["page_table"],
                           pos_begin=32, pos_end=P)
    torch.cuda.synchronize()
    j = np.arange(32, P)
    k = host(d["k_index_pool"])[h["page_table"][j // 64], j % 64]
    q = host(d["q_index"])
    want = sum(h["w_index"][:, i, None].astype(np.float64) * np.maximum(q[:, i] @ k.T, 0)
               for i in range(heads))
    assert rel_l2(host(s), want) <= 1e-6   # fp32 sums of exact products


@pytest.mark.parametrize("page", [4, 8, 16])
@pytest.mark.parametrize("R", [15, 77], ids=["few_rows", "more_rows"])
def test_bf16_short_pages(page, R):
    """Pages shorter than a key tile: a wave's rows in one page (8 and 16), or a
    lookup per row (4).  Splits and ranges begin and end inside pages, tiles and
    waves' rows; the last ones hold 1, 5 and 9 keys of a tile."""
    from paper_2607_14952_amd import inputs
    from paper_2607_14952_amd.replay import device_inputs
    from tests.test_gpu_parity import check_backward, check_forward
    cfg = _bf16(f"page{page}_r{R}", 1_003, R, page=page)
    h = inputs.dense_inputs(cfg)
    dev = device_inputs(h)
    P = cfg.prefix_len
    splits = [(0, 32), (32, 33), (33, 69), (69, 500), (500, 521), (521, 1_001), (1_001, P),
              (P, P + 7), (P + 7, P + R)]
    out, lse, o_ref, l_ref = check_forward(cfg, h, dev, splits, P=P, q_pos0=P)
    check_backward(cfg, h, dev, out, lse, o_ref, l_ref,
                   [(0, 41), (41, 42), (42, 777), (777, P + 5), (P + 5, P + R)], P=P, q_pos0=P)


@pytest.mark.parametrize("cfg,cuts", [
    (_bf16("ranges_few", 4_100, 20), [0, 1_000, 1_000, 1_033, 2_500, 4_100, 4_120]),
    (_bf16("ranges_many", 3_000, 3), list(range(0, 3_003, 77)) + [3_003]),
    (_bf16("ranges_whole", 600, 2_100), [0, 300, 600, 2_700]),
    (_f32("ranges", 4, 2, 64, 64, 6_000, 40), [0, 2_000, 2_100, 6_000, 6_040]),
    (_f32("ranges_generic", 2, 1, 160, 160, 300, 9), [0, 100, 300, 309]),
    # ranges of a few keys, which run on the generic kernels between others
    (_f32("ranges_small", 4, 2, 64, 64, 600, 4), [0, 5, 300, 306, 600, 604]),
], ids=lambda x: getattr(x, "name", ""))
def test_bwd_ranges_equal_calls(cfg, cuts):
    """Ranges that share launches leave the bits of one call per range: several
    chunks each, more ranges than one launch takes, an empty one, ranges whose
    one chunk fills the chip, and dq accumulated onto given values."""
    import torch

    from paper_2607_14952_amd import inputs
    from paper_2607_14952_amd.replay import device_inputs
    dev = device_inputs(inputs.dense_inputs(cfg))
    kv = B.PagedKV(dev["k_pool"], dev["v_pool"], dev["page_table"])
    P = cfg.prefix_len
    kw = dict(prefix_len=P, q_pos0=P, scale=cfg.scale)
    op, lp = B.prefix_attn_fwd(dev["q"], kv, [(0, cfg.kv_len)], **kw)
    out, lse = B.lse_merge(op, lp, out_dtype=dev["q"].dtype)
    ranges = list(zip(cuts, cuts[1:]))
    print(f"[gpu] bwd ranges {cfg.name}", flush=True)
    for first in (0, B.FLAG_ACCUMULATE_DQ):
        start = torch.ones((cfg.resp_len, cfg.n_q_heads, cfg.head_dim), device="cuda")
        dq, dk, dv = start.clone(), None, None
        for r, (b, e) in enumerate(ranges):
            dq, dk, dv = B.prefix_attn_bwd(dev["q"], kv, dev["d_out"], out, lse, kv_begin=b,
                                           kv_end=e, dq=dq, dk_resp=dk, dv_resp=dv,
                                           flags=B.FLAG_ACCUMULATE_DQ if r else first, **kw)
        got = B.prefix_attn_bwd_ranges(dev["q"], kv, dev["d_out"], out, lse, ranges,
                                       dq=start.clone(), flags=first, **kw)
        torch.cuda.synchronize()
        for x, y in zip((dq, dk, dv), got):
            assert torch.equal(x, y)


@pytest.mark.parametrize("cfg,begin", [
    # whole rounds of row tiles in two chunks, one tile a KV head (the last 64 packed
    # rows, or 16 tokens of 32 heads) in many
    (_bf16("tail_r1036", 9_600, 1_036), 17),
    (_bf16("tail_g16", 7_000, 514, hq=32), 3),
    # in one chunk, which writes its result itself
    (_bf16("tail_r2056", 1_500, 2_056), 17),
    (_bf16("tail_g1", 1_000, 8_200, hq=4, hkv=4), 0),
    (_bf16("tail_half", 1_200, 3_000, page=8), 5),
], ids=lambda x: getattr(x, "name", ""))
def test_dq_tail(cfg, begin):
    """A range whose last row tiles are cut into more key chunks than the others,
    against ranges of seven key tiles, which are never cut.  P and dS are formed key
    by key, so that only the order of the fp32 additions differs: under 1,000 of
    them per element, 2^-24 of the running sum each (6e-5; 1e-6 where they fall at
    random)."""
    import torch

    from paper_2607_14952_amd import inputs
    from paper_2607_14952_amd.replay import device_inputs
    dev = device_inputs(inputs.dense_inputs(cfg))
    kv = B.PagedKV(dev["k_pool"], dev["v_pool"], dev["page_table"])
    P, n = cfg.prefix_len, cfg.kv_len
    kw = dict(prefix_len=P, q_pos0=P, scale=cfg.scale)
    op, lp = B.prefix_attn_fwd(dev["q"], kv, [(0, n)], **kw)
    out, lse = B.lse_merge(op, lp, out_dtype=dev["q"].dtype)
    print(f"[gpu] dq tail {cfg.name}", flush=True)
    cuts = [begin, *range((begin // 32 + 7) * 32, n, 224), n]
    for flags in (0, B.FLAG_ACCUMULATE_DQ):
        start = torch.full((cfg.resp_len, cfg.n_q_heads, cfg.head_dim), 0.5, device="cuda")
        want, _, _ = B.prefix_attn_bwd_ranges(dev["q"], kv, dev["d_out"], out, lse,
                                              list(zip(cuts, cuts[1:])), dq=start.clone(),
                                              flags=flags, **kw)
        got, _, _ = B.prefix_attn_bwd(dev["q"], kv, dev["d_out"], out, lse, kv_begin=begin,
                                      kv_end=n, dq=start.clone(), flags=flags, **kw)
        torch.cuda.synchronize()
        assert (got - want).abs().max().item() <= 2e-5 * want.abs().max().item()


@pytest.mark.parametrize("page,prefix,backward", [(16, 16 * 61 + 5, True), (16, 16 * 64, False),
                                                  (64, 64 * 37 + 1, True), (32, 32 * 9, True)])
def test_cyclic_replay_pages(page, prefix, backward):
    """Cyclic shards through one table (pages of a key tile or more) and through
    a table each (shorter ones), with and without a partly filled last page."""
    import torch

    import oracle as O
    from paper_2607_14952_amd import inputs
    from paper_2607_14952_amd.replay import ReplayStep, device_inputs
    from tests._gpu import TOL_BF16, host, lse_err, rel_l2
    cfg = _bf16(f"cyclic_p{page}", prefix, 21, page=page, shards=5, ownership="cyclic",
                backward=backward)
    h = inputs.dense_inputs(cfg)
    step = ReplayStep(cfg, device_inputs(h))
    print(f"[gpu] {cfg.name}", flush=True)
    step.step()
    torch.cuda.synchronize()
    kw = dict(page_size=page, q_pos0=cfg.q_pos0, scale=cfg.scale)
    o, l = O.attn_fwd(h["q"], h["k_pool"], h["v_pool"], h["page_table"], **kw)
    assert rel_l2(host(step.out), o) <= TOL_BF16["out"]
    assert lse_err(host(step.lse), l) <= TOL_BF16["lse"]
    for c in range(cfg.n_shards):
        pos = O.cyclic_owned_positions(prefix, page, cfg.n_shards, c)
        so, sl = O.attn_fwd(h["q"], h["k_pool"], h["v_pool"], h["page_table"], key_positions=pos, **kw)
        assert rel_l2(host(step.shard_out[c]), so) <= TOL_BF16["out"]
        assert lse_err(host(step.shard_lse[c]), sl) <= TOL_BF16["lse"]
    if backward:
        refs = O.attn_bwd(h["q"], h["k_pool"], h["v_pool"], h["page_table"], h["d_out"],
                          prefix_len=prefix, out=o, lse=l, **kw)
        for got, ref in zip((step.dq, step.dk, step.dv), refs):
            assert rel_l2(host(got), ref) <= TOL_BF16["grad"]


@pytest.mark.parametrize("page", [16, 64])
def test_cyclic_shards_by_hand(page):
    """The shards of a cyclic step, called one by one through the stores and ranges that
    it names, leave its parts and its gradients, to the bit."""
    import torch

    from paper_2607_14952_amd import inputs
    from paper_2607_14952_amd.replay import ReplayStep, device_inputs
    cfg = _bf16(f"cyclic_hand_p{page}", page * 37 + 1, 21, page=page, shards=5, ownership="cyclic")
    dev = device_inputs(inputs.dense_inputs(cfg))
    step = ReplayStep(cfg, dev)
    print(f"[gpu] {cfg.name}", flush=True)
    step.step()
    kw = dict(prefix_len=cfg.prefix_len, q_pos0=cfg.q_pos0, scale=cfg.scale)
    dq = dk = dv = None
    for s, (b, e) in enumerate(step.shards):
        i, j = step.groups[s]
        o, l = B.prefix_attn_fwd(dev["q"], step.shard_kv[s], step.shard_splits[s], **kw)
        torch.cuda.synchronize()
        assert torch.equal(o, step.out_part[i:j]) and torch.equal(l, step.lse_part[i:j])
        dq, dk, dv = B.prefix_attn_bwd(dev["q"], step.shard_kv[s], dev["d_out"], step.out, step.lse,
                                       kv_begin=b, kv_end=e, dq=dq, dk_resp=dk, dv_resp=dv,
                                       flags=B.FLAG_ACCUMULATE_DQ if s else 0, **kw)
    torch.cuda.synchronize()
    for x, y in zip((dq, dk, dv), (step.dq, step.dk, step.dv)):
        assert torch.equal(x, y)


@pytest.mark.parametrize("d", [64, 160], ids=["matrix_cores", "generic"])
def test_f32_backward_in_less_workspace(d):
    """An fp32 backward also runs in the workspace of a block with fewer response keys,
    and in one that holds no more than Delta and the log-normalizers."""
    import torch

    from paper_2607_14952_amd import inputs
    from paper_2607_14952_amd.replay import device_inputs
    from tests._gpu import TOL_F32, host, rel_l2
    cfg = _f32(f"workspace_d{d}", 6, 2, d, d, 300, 40)
    dev = device_inputs(inputs.dense_inputs(cfg))
    kv = B.PagedKV(dev["k_pool"], dev["v_pool"], dev["page_table"])
    P, q0, n = cfg.prefix_len, cfg.prefix_len + 21, 19
    q, d_out = dev["q"][21:], dev["d_out"][21:]
    kw = dict(prefix_len=P, q_pos0=q0, scale=cfg.scale)
    op, lp = B.prefix_attn_fwd(q, kv, [(0, q0 + n)], **kw)
    out, lse = B.lse_merge(op, lp)
    want = B.prefix_attn_bwd(q, kv, d_out, out, lse, **kw)
    stat = -(-n * cfg.n_q_heads * 4 // 256) * 256
    for ws in (B.bwd_workspace(q, kv, prefix_len=P, q_pos0=P),
               torch.empty(2 * stat, dtype=torch.uint8, device="cuda")):
        print(f"[gpu] f32 backward d={d} in {ws.numel()} bytes", flush=True)
        got = B.prefix_attn_bwd(q, kv, d_out, out, lse, workspace=ws, **kw)
        torch.cuda.synchronize()
        for x, y in zip(got, want):
            assert rel_l2(host(x), host(y)) <= TOL_F32["grad"]
    with pytest.raises(B.LongStrawError) as ei:
        B.prefix_attn_bwd(q, kv, d_out, out, lse, workspace=ws[:2 * stat - 256], **kw)
    assert ei.value.name == "LS_ERR_WORKSPACE"


@pytest.mark.parametrize("bad", [float("nan"), float("inf")], ids=["nan", "inf"])
@pytest.mark.parametrize("hq,d,dv,resp", [(4, 64, 64, 40), (6, 128, 96, 150), (6, 40, 72, 40)],
                         ids=["d64", "four_groups", "d40"])
def test_f32_rows_before_a_bad_position(hq, d, dv, resp, bad):
    """A response position whose key and value are not finite reaches the rows that see
    it, not those before it in the same tiles; a row whose query and d_out are not
    reaches the keys that it sees, not those after it."""
    import numpy as np
    import torch

    from paper_2607_14952_amd import inputs
    from paper_2607_14952_amd.replay import device_inputs
    from tests._gpu import TOL_F32, host, rel_l2
    cfg = _f32(f"bad_d{d}", hq, 2, d, dv, 4_103 if resp > 100 else 70, resp)
    dev = device_inputs(inputs.dense_inputs(cfg))
    P, R = cfg.prefix_len, cfg.resp_len
    kw = dict(prefix_len=P, q_pos0=P, scale=cfg.scale)

    def run(t):
        kv = B.PagedKV(t["k_pool"], t["v_pool"], t["page_table"])
        op, lp = B.prefix_attn_fwd(t["q"], kv, [(0, P // 2), (P // 2, P + R)], **kw)
        out, lse = B.lse_merge(op, lp)
        dq = torch.full((R, hq, d), 0.5, device="cuda")
        _, dk, dv = B.prefix_attn_bwd(t["q"], kv, t["d_out"], out, lse, dq=dq,
                                      flags=B.FLAG_ACCUMULATE_DQ, **kw)
        torch.cuda.synchronize()
        return [host(x) for x in (out, lse.t(), dq, dk, dv)]

    good = run(dev)
    at = R - 15
    page, slot = int(dev["page_table"][(P + at) // cfg.page_size]), (P + at) % cfg.page_size
    t = {k: v.clone() for k, v in dev.items()}
    t["k_pool"][page, slot] = bad
    t["v_pool"][page, slot] = bad
    print(f"[gpu] {cfg.name}: key and value {bad}", flush=True)
    got = run(t)
    for x, y in zip(got[:3], good):
        assert np.isfinite(x[:at]).all() and rel_l2(x[:at], y[:at]) <= TOL_F32["grad"]
    for x in (got[0], got[2]):
        assert not np.isfinite(x[at:]).all(axis=(1, 2)).any()
    t = {k: v.clone() for k, v in dev.items()}
    t["q"][at] = bad
    t["d_out"][at] = bad
    print(f"[gpu] {cfg.name}: query and d_out {bad}", flush=True)
    got = run(t)
    for x, y in zip(got[:3], good):
        rest = np.arange(R) != at
        assert np.isfinite(x[rest]).all() and rel_l2(x[rest], y[rest]) <= TOL_F32["grad"]
    for x, y in zip(got[3:], good[3:]):
        assert np.isfinite(x[at + 1:]).all() and rel_l2(x[at + 1:], y[at + 1:]) <= TOL_F32["grad"]
        assert not np.isfinite(x[:at + 1]).all(axis=(1, 2)).any()


@pytest.mark.parametrize("cfg", [_bf16("splits_bf16", 3_603, 21), _bf16("splits_p4", 3_603, 9, page=4),
                                 _f32("splits_f32", 4, 2, 64, 64, 3_603, 21),
                                 _f32("splits_generic", 2, 1, 160, 160, 3_603, 5)],
                         ids=lambda c: c.name)
def test_more_splits_than_one_launch_takes(cfg):
    """About 900 splits of a few keys, in three launches: the second and third have a
    base and parts of their own, and the response's split is in the third."""
    from paper_2607_14952_amd import inputs
    from paper_2607_14952_amd.replay import device_inputs
    from tests.test_gpu_parity import check_forward
    h = inputs.dense_inputs(cfg)
    P = cfg.prefix_len
    splits = [(b, min(b + 4, P)) for b in range(0, P, 4)] + [(P, P + cfg.resp_len)]
    assert len(splits) > 2 * 448
    check_forward(cfg, h, device_inputs(h), splits, P=P, q_pos0=P)


@pytest.mark.parametrize("page", [8, 16])
@pytest.mark.parametrize("R,P,n", [(77, 4_096, 3), (512, 8_192, 8), (300, 3, 1)],
                         ids=["four_waves", "eight_waves", "own_keys"])
def test_short_pages_leave_the_bits_of_long_ones(page, R, P, n):
    """Pages of 8 and 16 take workgroups of four or eight waves by the splits' lengths and
    number; either way each row's partial results are those of the same positions in
    pages of 64."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(page + R)
    total = -(-(P + R) // 64) * 64
    k, v = (torch.randn((total, 2, 256), device="cuda", generator=g).to(torch.bfloat16)
            for _ in range(2))
    q = torch.randn((R, 16, 256), device="cuda", generator=g).to(torch.bfloat16)
    splits = [(P * i // n, P * (i + 1) // n) for i in range(n)] + [(P, P + R)]
    print(f"[gpu] pages of {page}, R={R}", flush=True)
    got = []
    for S in (page, 64):
        table = torch.randperm(total // S, device="cuda", generator=g)
        pools = [torch.empty_like(x).view(-1, S, 2, 256) for x in (k, v)]
        for pool, x in zip(pools, (k, v)):
            pool[table] = x.view(-1, S, 2, 256)
        got.append(B.prefix_attn_fwd(q, B.PagedKV(*pools, table.to(torch.int32)), splits,
                                     prefix_len=P, q_pos0=P, scale=1 / 16))
    torch.cuda.synchronize()
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
