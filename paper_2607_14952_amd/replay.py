"""One response-replay step over a paged prefix, composed from the library calls.

forward  : every split's local (o_r, l_r)        -> ls_prefix_attn_fwd (one launch)
           splits of a shard -> shard (o_s, l_s)  -> ls_lse_merge_groups (one launch;
           shards + response -> global (o, l)        fp32 per shard, q dtype for the
           result; with bf16_numerator the last numerator is reduced in bf16, as
           the production composition noted after Eq. qwen-global-attn)
           (the single-GPU form of the cross-rank merge, Eq. qwen-lse-parts and
           Eq. qwen-global-attn)
backward : ls_prefix_attn_bwd_ranges over the shards' key ranges, dq accumulated
           in shard order (Eq. qwen-dq-reduce);
           the response range also yields the response dK/dV (lazy gradient pages:
           prefix keys get none).

Shards own contiguous prefix ranges, or, with ``ownership="cyclic"``, the pages
p with p mod n_shards = c (Eq. qwen-page-owner).  A cyclic step reads the store
through a table of its own that names the prefix pages shard by shard, so that
each shard's keys form one range of it.  Renumbering is exact here because every
prefix position precedes every query row, so each prefix key is visible to each
row whatever its position; the shard that owns a partly filled last page comes
last, which keeps that page in its place before the response's positions.  With
pages shorter than a key tile a shard's range might begin inside a tile of that
table, which would round its results differently from a shard's own store: such
a step keeps a table and a launch per shard.
"""
from __future__ import annotations

import numpy as np

from . import binding as B


def to_device(arr: np.ndarray, device="cuda"):
    """numpy input (uint16 bf16 bit patterns, float32 or int32) -> torch device tensor."""
    import torch
    if arr.dtype == np.uint16:
        return torch.from_numpy(arr.view(np.int16)).view(torch.bfloat16).to(device)
    return torch.from_numpy(np.ascontiguousarray(arr)).to(device)


def device_inputs(host: dict, device="cuda") -> dict:
    out = {}
    for k in ("q", "k_pool", "v_pool", "page_table", "d_out", "latent_pool", "idx"):
        if k in host:
            out[k] = to_device(host[k], device)
    return out


def cyclic_shards(cfg):
    """Cyclic ownership: the ranges of the shards that own positions (in shard
    order, then the response's) in a table that names the prefix pages shard by
    shard, and that table's prefix pages (logical page numbers, in table order).
    A partly filled last page stays last, so the shard that owns it comes last
    in the table."""
    owners = [c for c in range(cfg.n_shards) if cfg.shard_len(c)]
    last = (cfg.n_prefix_pages - 1) % cfg.n_shards
    in_table = owners
    if cfg.prefix_len % cfg.page_size:
        in_table = [c for c in owners if c != last] + [last]
    start, order = {}, []
    for c in in_table:
        start[c] = len(order) * cfg.page_size
        order += cfg.shard_pages(c)
    shards = [(start[c], start[c] + cfg.shard_len(c)) for c in owners]
    return shards + [(cfg.prefix_len, cfg.kv_len)], order


_CUS = 256
_PIECES = (1, 2, 3, 4, 5, 6, 8, 10, 12, 16, 24, 32, 48, 64)   # of a split


def fine_splits(cfg, splits, n_rows=None):
    """The shards' splits (lists of key ranges, the response's list last), each cut
    into the number of equal pieces that makes the forward and merge of n_rows
    (default: the response's) tokens shortest.

    A bf16 workgroup takes 32-key tiles of one split for 256 packed query rows
    (128 where there are no more) and one runs per CU, so a launch takes
    ceil(workgroups / 256) rounds of a split's tiles plus about 6 for its start
    and end, and one more short round where the response's workgroups find no
    idle CU.  In fp32, 128 rows a workgroup, two share a CU at 1.6 times the time,
    or, where those would not fill the CUs once, 32 rows whose four waves share the
    tiles.  Each further part is written and read once more: 0.41 ns per KiB row
    (1,111 rows, 33 -> 65 parts: +241 us).

    Measured, whole -> cut: bf16, 1 row x 131,075 keys in 64 splits 72 -> 64 us (2
    pieces), 16 rows x 262,144 keys in 32 splits 248 -> 137 us (4), 150 rows x 1M
    3,071 -> 2,276 us (4); fp32, 1 row x 30,000 keys in 2 splits 873 -> 56 us
    (32), 128 rows x 4,096 in 2 66 -> 32 (8); capture of 30,000 positions in chunks
    of 1,024 17.9 -> 7.6 ms, of 100,000 93 -> 72 ms.  77 rows x 262,144 (198 workgroups)
    gain nothing (421, 434, 430 us for 1, 2, 4), so a cut must promise 8%; 4,096
    rows fill 33 rounds and stay whole."""
    tokens = cfg.resp_len if n_rows is None else n_rows
    rows = tokens * cfg.group
    prefix = [r for sp in splits[:-1] for r in sp]
    n, hkv = len(prefix), cfg.n_kv_heads
    if not prefix or -(-rows // 256) * hkv * n >= 4 * _CUS:
        return splits   # four rounds or more: nothing to gain
    tiles = -(-max(e - b for b, e in prefix) // 32)

    if cfg.dtype == "f32":
        tile_ns = 4000 * max(cfg.head_dim, cfg.head_dim_v) / 128

        def launch(f):
            wide = -(-rows // 128) * hkv * n * f
            if wide >= _CUS:
                return -(-wide // (2 * _CUS)) * 1.6 * (-(-tiles // f) + 3)
            return -(-(-(-rows // 32) * hkv * n * f) // _CUS) * (-(-tiles // (4 * f)) + 4)
    else:
        per_wg = 256 if cfg.page_size >= 8 and rows > 128 else 128
        tile_ns = 1600 if per_wg == 256 else 950

        def launch(f):
            own = -(-rows // per_wg) * hkv   # workgroups of one split
            rounds = -(-own * n * f // _CUS)
            late = 0
            if rounds * _CUS - own * n * f < own:
                late = 6 + min(tiles, -(-tokens // 32))
            return rounds * (-(-tiles // f) + 6) + late

    part = 0.41 / tile_ns * tokens * cfg.n_q_heads * cfg.head_dim_v / 256 * n

    def cost(f):
        return launch(f) + part * f

    most = max(1, min(64, tiles // 8, 1024 // n))
    f = min((x for x in _PIECES if x <= most), key=cost)
    if cost(f) > 0.92 * cost(1):
        return splits

    def cut(b, e):
        lo = b // 32 * 32   # pieces begin with a tile
        step = -(-(e - lo) // (32 * f)) * 32
        return [(max(b, x), min(e, x + step)) for x in range(lo, e, step)]

    return [[p for r in sp for p in cut(*r)] for sp in splits[:-1]] + splits[-1:]


class ReplayStep:
    """Buffers and call sequence of one fwd(+bwd) replay over a config's shards.

    shards[s] is shard s's key range and splits[i] that of part i (out_part[i],
    lse_part[i]; shard s has parts groups[s] and the ranges shard_splits[s]), as
    shard_kv[s] names positions: a cyclic shard's store has its owned pages first,
    so that its keys are 0 .. shard_len - 1.  Forward-only and fp32 steps have more
    parts than configured splits (fine_splits)."""

    def __init__(self, cfg, dev: dict, *, backward: bool | None = None, stream=None):
        import torch
        self.cfg = cfg
        self.dev = dev
        self.kv = B.PagedKV(dev["k_pool"], dev["v_pool"], dev["page_table"])
        self.backward_enabled = cfg.backward if backward is None else backward
        self.stream = stream
        self._shard_kv = None
        q = dev["q"]
        R, Hq, D, Dv = cfg.resp_len, cfg.n_q_heads, cfg.head_dim, cfg.head_dim_v
        own = (cfg.prefix_len, cfg.kv_len)
        self.cyclic = cfg.ownership == "cyclic"
        if self.cyclic:
            self._table = dev["page_table"].cpu().numpy()
            owners = [c for c in range(cfg.n_shards) if cfg.shard_len(c)]
            splits = [cfg.virtual_splits(c) for c in owners] + [[own]]
            self.shards = [(0, cfg.shard_len(c)) for c in owners] + [own]
            if cfg.page_size >= 32:
                self._ranges, order = cyclic_shards(cfg)
                self.stores = [self._store(order)]
            else:
                self._ranges = self.shards
                self._shard_kv = self.stores = self._shard_stores()
        else:
            self.shards = self._ranges = [r for r in cfg.shard_ranges() if r[0] < r[1]]
            self.stores = [self.kv]
            every = [r for r in cfg.splits() if r[0] < r[1]]
            splits = [[r for r in every if b <= r[0] and r[1] <= e] for b, e in self.shards]
            assert sum(map(len, splits)) == len(every)
        # where each shard's own coordinates begin in its store
        base = [r[0] - o[0] for r, o in zip(self._ranges, self.shards)]
        splits = [[(x + i, x + j) for i, j in sp] for x, sp in zip(base, splits)]
        # With a bf16 backward the splits stay as configured: other ones round P, and
        # with it the bf16 output inside Delta, in other places, which moves the dq of
        # a few rows with concentrated probabilities by up to 1.3e-2 (10 rows x 33,374
        # keys, one in 100 aimed at a row; both results are as far from 64 bits).
        if len(self.stores) == 1 and (cfg.dtype == "f32" or not self.backward_enabled):
            splits = fine_splits(cfg, splits)
        # The parts in launch order (key order of one store, else shard by shard);
        # shard s has the parts groups[s] and is launched from store_of(s).
        order = sorted(range(len(splits)), key=lambda s: splits[s]) \
            if len(self.stores) == 1 else range(len(splits))
        self._launch, self.splits, self.groups = [], [], [None] * len(splits)
        for s in order:
            self.groups[s] = (len(self.splits), len(self.splits) + len(splits[s]))
            self._launch += splits[s]
            self.splits += [(i - base[s], j - base[s]) for i, j in splits[s]]
        self.shard_splits = [self.splits[i:j] for i, j in self.groups]
        kw = dict(dtype=torch.float32, device=q.device)
        self.out_part = torch.empty((len(self.splits), R, Hq, Dv), **kw)
        self.lse_part = torch.empty((len(self.splits), Hq, R), **kw)
        self.shard_out = torch.empty((len(self.shards), R, Hq, Dv), **kw)
        self.shard_lse = torch.empty((len(self.shards), Hq, R), **kw)
        self.out = torch.empty((R, Hq, Dv), dtype=q.dtype, device=q.device)
        self.lse = torch.empty((Hq, R), **kw)
        if self.backward_enabled:
            self.dq = torch.empty((R, Hq, D), **kw)
            self.dk = torch.zeros((cfg.kv_len - cfg.prefix_len, cfg.n_kv_heads, D), **kw)
            self.dv = torch.zeros((cfg.kv_len - cfg.prefix_len, cfg.n_kv_heads, Dv), **kw)
            self.ws = B.bwd_workspace(q, self.kv, prefix_len=cfg.prefix_len, q_pos0=cfg.q_pos0)

    def _store(self, pages):
        """A store whose first pages are these (logical pages of the step's table)."""
        import torch
        t = self._table.copy()
        t[:len(pages)] = self._table[pages]
        return B.PagedKV(self.dev["k_pool"], self.dev["v_pool"],
                         torch.from_numpy(t).to(self.dev["page_table"].device))

    def _shard_stores(self):
        cfg = self.cfg
        return [self._store(cfg.shard_pages(c)) for c in range(cfg.n_shards)
                if cfg.shard_len(c)] + [self.kv]

    @property
    def shard_kv(self):
        """Each shard's own store (made when first asked for where the step itself
        reads all cyclic shards through one)."""
        if self._shard_kv is None:
            self._shard_kv = self._shard_stores() if self.cyclic else [self.kv] * len(self.shards)
        return self._shard_kv

    def store_of(self, s: int):
        """The store that the step launches shard s from."""
        return self.stores[s if len(self.stores) > 1 else 0]

    def forward_splits(self):
        """Local (o_r, l_r) of every split, one launch per store."""
        c = self.cfg
        kw = dict(prefix_len=c.prefix_len, q_pos0=c.q_pos0, scale=c.scale, stream=self.stream)
        if len(self.stores) == 1:
            B.prefix_attn_fwd(self.dev["q"], self.stores[0], self._launch, out_part=self.out_part,
                              lse_part=self.lse_part, **kw)
            return
        for s, (i, j) in enumerate(self.groups):
            B.prefix_attn_fwd(self.dev["q"], self.stores[s], self._launch[i:j],
                              out_part=self.out_part[i:j], lse_part=self.lse_part[i:j], **kw)

    def merge(self):
        """Splits -> per-shard results (fp32) -> global result (q dtype)."""
        flags = B.FLAG_BF16_NUMERATOR if self.cfg.bf16_numerator else 0
        if len(self.groups) <= B.MAX_MERGE_GROUPS:
            B.lse_merge_groups(self.out_part, self.lse_part, self.groups, group_out=self.shard_out,
                               group_lse=self.shard_lse, out=self.out, lse=self.lse, flags=flags,
                               stream=self.stream)
            return
        for s, (i, j) in enumerate(self.groups):
            B.lse_merge(self.out_part[i:j], self.lse_part[i:j], out=self.shard_out[s],
                        lse=self.shard_lse[s], stream=self.stream)
        B.lse_merge(self.shard_out, self.shard_lse, out=self.out, lse=self.lse, flags=flags,
                    stream=self.stream)

    def forward(self):
        self.forward_splits()
        self.merge()
        return self.out, self.lse

    def backward_range(self, r: int):
        """dq contribution of shard range r (accumulated after the first range);
        the response range also writes the response dK/dV.  Ranges after the
        first reuse the Delta and lse * log2(e) the first one left in the
        workspace, so ranges must run in order, starting at 0."""
        c = self.cfg
        b, e = self._ranges[r]
        B.prefix_attn_bwd(self.dev["q"], self.store_of(r), self.dev["d_out"], self.out, self.lse,
                          prefix_len=c.prefix_len, q_pos0=c.q_pos0, scale=c.scale,
                          kv_begin=b, kv_end=e,
                          flags=(B.FLAG_ACCUMULATE_DQ | B.FLAG_PREP_READY) if r > 0 else 0,
                          dq=self.dq, dk_resp=self.dk, dv_resp=self.dv, workspace=self.ws,
                          stream=self.stream)

    def backward(self):
        """Every shard range, in one call per store: what backward_range leaves after the
        last."""
        c = self.cfg
        if len(self.stores) > 1:
            for r in range(len(self.shards)):
                self.backward_range(r)
            return self.dq, self.dk, self.dv
        B.prefix_attn_bwd_ranges(self.dev["q"], self.stores[0], self.dev["d_out"], self.out, self.lse,
                                 self._ranges, prefix_len=c.prefix_len, q_pos0=c.q_pos0,
                                 scale=c.scale, dq=self.dq, dk_resp=self.dk, dv_resp=self.dv,
                                 workspace=self.ws, stream=self.stream)
        return self.dq, self.dk, self.dv

    def step(self):
        self.forward()
        if self.backward_enabled:
            self.backward()
