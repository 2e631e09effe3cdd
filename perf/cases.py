"""Cases that stand for the framework's use, to be timed and checked on one GPU.

``listed()`` names the fixed ones, ``draw(rng)`` makes more of the same ranges.
A case is a dict of plain values; ``prepare(case, seed)`` draws its inputs on
the GPU and builds what a program keeps between calls (step objects, pools,
workspaces), ``run(state)`` makes one pass through the public entry points, and
``exact(case, seed)`` computes the same outputs in 64 bits with plain torch.

Kinds:
  replay     one response replayed against a paged prefix (ReplayStep): split
             forward, LSE merges and, with ``bwd``, dq per shard and the
             response dK/dV.  fp32 or bf16 store; contiguous or cyclic page
             ownership; bf16 or fp32 numerator in the cross-shard merge.
  blockwise  one member of a group replayed block by block in reverse against a
             resident prefix (append, forward, backward, pop).
  capture    no-grad capture of a prompt, chunk by chunk (append + prefill).
  sparse     MLA replay over selected latent rows plus the response window.
  dsa        index scores over the prefix and each row's top-k.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2607_14952_amd import binding as B
from paper_2607_14952_amd.blockwise import BlockwiseReplay, ResidentPrefix
from paper_2607_14952_amd.capture import PrefixCapture
from paper_2607_14952_amd.configs import CaptureConfig, ReplayConfig
from paper_2607_14952_amd.dsa import DsaSelect
from paper_2607_14952_amd.replay import ReplayStep

_DEV = "cuda"


# ------------------------------------------------------------------ cases
def _replay(dtype="bf16", hq=16, hkv=2, d=256, page=256, prefix=0, resp=0, shards=8, splits=4,
            bwd=True, cyclic=False, bf16num=False):
    return dict(kind="replay", dtype=dtype, hq=hq, hkv=hkv, d=d, page=page, prefix=prefix,
                resp=resp, shards=shards, splits=splits, bwd=bwd, cyclic=cyclic, bf16num=bf16num)


def listed():
    return [
        # the smallest configuration (c1): an fp32 replay of 128 tokens, where
        # launches and latency count
        dict(_replay("f32", 2, 1, 64, 64, 4096, 128, 2, 1), name="f32_tiny"),
        # an fp32 replay with grouped heads, as a numerics check of a real layer runs it;
        # ragged prefix and response
        dict(_replay("f32", 8, 2, 128, 64, 16_001, 500, 2, 4), name="f32_gqa"),
        # one decoded token against a captured prompt of ordinary length
        dict(_replay(prefix=131_075, resp=1, splits=8, bwd=False), name="decode_row_131k"),
        # 16 rows against the 2M store: page streaming, bound by HBM
        dict(_replay(prefix=2_097_152, resp=16, splits=32, bwd=False), name="decode_16_2m"),
        # a short response scored and differentiated against a long prompt
        dict(_replay(prefix=262_144, resp=77), name="short_262k"),
        # an ordinary response with the production composition: cyclic pages of
        # 64 positions and the bf16 numerator
        dict(_replay(prefix=100_003, resp=1_111, page=64, cyclic=True, bf16num=True),
             name="cyclic_100k"),
        # the headline step (c3): 4,096 tokens against 2,097,152 positions
        dict(_replay(prefix=2_097_152, resp=4_096), name="replay_2m"),
        # a group member in blocks of 2,048 tokens, the last one ragged (c4's shape, shorter)
        dict(kind="blockwise", prefix=262_144, resp=3_000, block=2_048, shards=8, splits=8,
             name="blockwise_262k"),
        # capture of a 64K prompt in 4,096-token chunks, a ragged one last
        dict(kind="capture", length=61_000, chunk=4_096, name="capture_61k"),
        # sparse MLA replay (c5): 2,048 tokens, 2,048 selected rows each
        dict(kind="sparse", prefix=2_097_152, resp=2_048, topk=2_048, name="sparse_2m"),
        # the same for a short response
        dict(kind="sparse", prefix=262_144, resp=24, topk=2_048, name="sparse_short"),
        # the selection that feeds it: 32 index heads
        dict(kind="dsa", prefix=524_288, resp=500, heads=32, topk=2_048, name="dsa_524k"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["f32", "decode", "replay", "replay", "replay", "blockwise", "capture",
                       "sparse", "sparse", "dsa"])
    if kind == "f32":
        hkv = rng.choice([1, 2, 3])
        hq = hkv * rng.choice([1, 2, 3, 4, 8])
        step = 4 // math.gcd(4, hq)   # a split's log-normalizers start on 16 bytes
        return _replay("f32", hq, hkv, rng.choice([64, 96, 128]), rng.choice([16, 32, 64]),
                       _log(rng, 500, 32_000), -(-_log(rng, 1, 600) // step) * step,
                       rng.choice([1, 2]), rng.choice([1, 4]))
    heads = rng.choice([(16, 2), (16, 2), (8, 2), (32, 2), (8, 1), (4, 4)])
    page = rng.choice([16, 64, 256, 256])
    if kind == "decode":
        prefix = _log(rng, 16_384, 2_097_152)
        return _replay(hq=heads[0], hkv=heads[1], page=page, prefix=prefix, resp=_log(rng, 1, 16),
                       splits=max(1, min(32, prefix // 16_384)), bwd=False)
    if kind == "replay":
        while True:
            prefix, resp = _log(rng, 2_048, 2_097_152), _log(rng, 4, 4_096)
            if prefix * resp * heads[0] <= 2_097_152 * 4_096 * 16 // 3:   # a third of the headline
                break
        cyclic = rng.random() < 0.3
        return _replay(hq=heads[0], hkv=heads[1], page=page, prefix=prefix, resp=resp,
                       shards=rng.choice([1, 2, 8, 8]), splits=rng.choice([2, 4, 4]),
                       cyclic=cyclic, bf16num=rng.random() < 0.3, bwd=rng.random() < 0.8)
    if kind == "blockwise":
        return dict(kind=kind, prefix=_log(rng, 32_768, 524_288) // 256 * 256,
                    resp=_log(rng, 600, 6_000), block=rng.choice([512, 1_024, 2_048]), shards=8,
                    splits=rng.choice([4, 8]))
    if kind == "capture":
        return dict(kind=kind, length=_log(rng, 3_000, 131_072),
                    chunk=rng.choice([1_024, 2_048, 4_096]))
    if kind == "sparse":
        return dict(kind=kind, prefix=_log(rng, 8_192, 2_097_152), resp=_log(rng, 1, 2_048),
                    topk=rng.choice([256, 1_024, 2_048, 2_048]))
    return dict(kind=kind, prefix=_log(rng, 8_192, 1_048_576), resp=_log(rng, 1, 512),
                heads=rng.choice([8, 16, 32, 32]), topk=rng.choice([256, 1_024, 2_048]))


# ------------------------------------------------------------------ inputs
class _Rand:
    """Seeded normals on the GPU (one generator per case and seed)."""

    def __init__(self, seed):
        self.g = torch.Generator(device=_DEV).manual_seed(seed)
        self.host = torch.Generator().manual_seed(seed)

    def normal(self, *shape, dtype=torch.bfloat16):
        return torch.randn(shape, dtype=dtype, device=_DEV, generator=self.g)

    def ints(self, n, hi):
        return torch.randint(0, hi, (n,), device=_DEV, generator=self.g)

    def table(self, n):
        return torch.randperm(n, generator=self.host).to(torch.int32).to(_DEV)


def _plant(r, k_pool, table, q, prefix, hkv):
    """1% of the prefix keys lean towards a response query, so that the
    probabilities of a row gather on some keys, as they do in a trained model."""
    n = prefix // 100
    if n == 0:
        return
    R, hq, _ = q.shape
    pos = torch.arange(n, device=_DEV) * 100 + r.ints(n, 100)   # distinct
    row, head = r.ints(n, R), r.ints(n, hq)
    S = k_pool.shape[1]
    page, slot, g = table[pos // S].long(), pos % S, head // (hq // hkv)
    k_pool[page, slot, g] = (k_pool[page, slot, g].float() + 4.0 * q[row, head].float()).to(
        k_pool.dtype)


def _replay_cfg(c):
    return ReplayConfig(name="case", seed=0, dtype=c["dtype"], n_q_heads=c["hq"],
                        n_kv_heads=c["hkv"], head_dim=c["d"], head_dim_v=c["d"],
                        page_size=c["page"], prefix_len=c["prefix"], resp_len=c["resp"],
                        n_shards=c["shards"], splits_per_shard=c["splits"], backward=c["bwd"],
                        ownership="cyclic" if c["cyclic"] else "contiguous",
                        bf16_numerator=c["bf16num"])


def _replay_inputs(c, seed):
    r = _Rand(seed)
    cfg = _replay_cfg(c)
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    # the response follows the prefix's last position, within its page where that has room
    n_pages = -(-cfg.kv_len // cfg.page_size)
    pool = (n_pages, cfg.page_size, cfg.n_kv_heads, cfg.head_dim)
    dev = dict(q=r.normal(cfg.resp_len, cfg.n_q_heads, cfg.head_dim, dtype=dt),
               k_pool=r.normal(*pool, dtype=dt), v_pool=r.normal(*pool, dtype=dt),
               page_table=r.table(n_pages),
               d_out=r.normal(cfg.resp_len, cfg.n_q_heads, cfg.head_dim, dtype=dt))
    _plant(r, dev["k_pool"], dev["page_table"], dev["q"], cfg.prefix_len, cfg.n_kv_heads)
    return cfg, dev


def _blockwise_inputs(c, seed):
    r = _Rand(seed)
    cfg = ReplayConfig(name="case", seed=0, dtype="bf16", n_q_heads=16, n_kv_heads=2, head_dim=256,
                       head_dim_v=256, page_size=256, prefix_len=c["prefix"], resp_len=c["resp"],
                       n_shards=c["shards"], splits_per_shard=c["splits"], table="sample",
                       pool_slack=1.125, block=c["block"])
    n_pre = cfg.n_prefix_pages
    n_phys = cfg.n_phys_pages
    perm = torch.randperm(n_phys, generator=r.host).to(torch.int32)
    pool = (n_phys, 256, 2, 256)
    store = dict(k_pool=r.normal(*pool), v_pool=r.normal(*pool), prefix_table=perm[:n_pre].to(_DEV),
                 free_pages=perm[n_pre:].sort().values)
    resp = dict(q=r.normal(cfg.resp_len, 16, 256), k=r.normal(cfg.resp_len, 2, 256),
                v=r.normal(cfg.resp_len, 2, 256), d_out=r.normal(cfg.resp_len, 16, 256))
    _plant(r, store["k_pool"], store["prefix_table"], resp["q"], cfg.prefix_len, 2)
    return cfg, store, resp


def _capture_inputs(c, seed):
    r = _Rand(seed)
    cfg = CaptureConfig(name="case", seed=0, n_q_heads=16, n_kv_heads=2, head_dim=256,
                        page_size=256, length=c["length"], chunk=c["chunk"])
    dev = dict(q_blocks=r.normal(cfg.n_chunks, cfg.chunk, 16, 256), k=r.normal(cfg.length, 2, 256),
               v=r.normal(cfg.length, 2, 256), page_table=r.table(cfg.n_logical_pages))
    return cfg, dev


def _sparse_inputs(c, seed):
    r = _Rand(seed)
    R, P, k = c["resp"], c["prefix"], min(c["topk"], c["prefix"])
    n_pages = -(-(P + R) // 64)
    d = dict(q=r.normal(R, 128, 576), pool=r.normal(n_pages, 64, 1, 576), table=r.table(n_pages),
             d_out=r.normal(R, 128, 512))
    # each row selects k distinct prefix positions, ascending: one per stratum
    edges = torch.arange(k + 1, dtype=torch.float64) * (P / k)
    lo = edges[:-1].ceil().long().to(_DEV)
    width = (edges[1:].ceil().long().to(_DEV) - lo).clamp(min=1)
    u = torch.rand((R, k), device=_DEV, generator=r.g, dtype=torch.float64)
    d["idx"] = (lo + torch.minimum((u * width).long(), width - 1)).to(torch.int32)
    return d


def _dsa_cfg(c):
    return ReplayConfig(name="case", seed=0, dtype="bf16", n_q_heads=128, n_kv_heads=1,
                        head_dim=576, head_dim_v=512, page_size=64, prefix_len=c["prefix"],
                        resp_len=c["resp"], sparse=True, topk=min(c["topk"], c["prefix"]),
                        index_heads=c["heads"])


def _dsa_inputs(c, seed):
    r = _Rand(seed)
    n_pages = -(-c["prefix"] // 64)
    return dict(q_index=r.normal(c["resp"], c["heads"], 128),
                w_index=r.normal(c["resp"], c["heads"], dtype=torch.float32)
                / math.sqrt(c["heads"]),
                k_index_pool=r.normal(n_pages, 64, 128), page_table=r.table(n_pages))


# ------------------------------------------------------------------ one pass
def prepare(case, seed):
    kind = case["kind"]
    if kind == "replay":
        cfg, dev = _replay_inputs(case, seed)
        return dict(kind=kind, step=ReplayStep(cfg, dev))
    if kind == "blockwise":
        cfg, store, resp = _blockwise_inputs(case, seed)
        host = {k: (t.view(torch.int16).cpu().numpy().view(np.uint16)
                    if t.dtype == torch.bfloat16 else t.cpu().numpy()) for k, t in store.items()}
        prefix = ResidentPrefix(cfg, host)
        return dict(kind=kind, replay=BlockwiseReplay(cfg, prefix), resp=resp)
    if kind == "capture":
        cfg, dev = _capture_inputs(case, seed)
        out = torch.empty((cfg.length, 16, 256), dtype=torch.bfloat16, device=_DEV)
        return dict(kind=kind, cap=PrefixCapture(cfg, dev), out=out)
    if kind == "sparse":
        d = _sparse_inputs(case, seed)
        kv = B.PagedKV(d["pool"], d["pool"], d["table"])
        R, P = case["resp"], case["prefix"]
        f32 = dict(dtype=torch.float32, device=_DEV)
        ws = B.sparse_workspace(d["q"], kv, d["idx"].shape[1], prefix_len=P, q_pos0=P,
                                backward=True)
        return dict(kind=kind, d=d, kv=kv, P=P, ws=ws, out=torch.empty((R, 128, 512), **f32),
                    lse=torch.empty((128, R), **f32), dq=torch.empty((R, 128, 576), **f32))
    return dict(kind=kind, sel=DsaSelect(_dsa_cfg(case), _dsa_inputs(case, seed)))


def run(state):
    kind = state["kind"]
    if kind == "replay":
        s = state["step"]
        s.step()
        if not s.backward_enabled:
            return dict(out=s.out, lse=s.lse)
        return dict(out=s.out, lse=s.lse, dq=s.dq, dk=s.dk, dv=s.dv)
    if kind == "blockwise":
        dq, dk, dv = state["replay"].run_member(state["resp"])
        return dict(dq=dq, dk=dk, dv=dv)
    if kind == "capture":
        cap, out = state["cap"], state["out"]
        for c in range(cap.cfg.n_chunks):
            b, e = cap.cfg.chunk_range(c)
            cap.chunk(c, out=out[b:e])
        return dict(out=out, k_pool=cap.k_pool, v_pool=cap.v_pool)
    if kind == "sparse":
        d, P = state["d"], state["P"]
        kw = dict(prefix_len=P, q_pos0=P, scale=576 ** -0.5, workspace=state["ws"])
        out, lse = B.sparse_attn_fwd(d["q"], state["kv"], d["idx"], out=state["out"],
                                     lse=state["lse"], **kw)
        dq = B.sparse_attn_bwd(d["q"], state["kv"], d["idx"], d["d_out"], out, lse,
                               dq=state["dq"], **kw)
        return dict(out=out, lse=lse, dq=dq)
    sel = state["sel"]
    idx = sel.run()
    return dict(idx=idx, idx_scores=sel.sel_scores, scores=sel.scores[:, :sel.cfg.prefix_len])


# ------------------------------------------------------------------ work and tolerance
def work(case):
    kind = case["kind"]
    if kind in ("replay", "blockwise"):
        if kind == "blockwise":
            case = _replay(prefix=case["prefix"], resp=case["resp"])
        R, P, hq, hkv, d = (case[k] for k in ("resp", "prefix", "hq", "hkv", "d"))
        es = 2 if case["dtype"] == "bf16" else 4
        pre, own = R * P, R * (R + 1) // 2
        flops = 4 * hq * d * (pre + own)
        nbytes = 2 * (P + R) * hkv * d * es + R * hq * (2 * d * es + 4)
        if case["bwd"]:
            flops += hq * d * (6 * pre + 10 * own)
            nbytes += R * hq * d * (es + 4) + 2 * R * hkv * d * 4
        return {"bytes": nbytes, "flops": flops}
    if kind == "capture":
        n = case["length"]
        return {"bytes": n * 256 * 2 * (2 * 16 + 4 * 2), "flops": 4 * 16 * 256 * (n * (n + 1) // 2)}
    if kind == "sparse":
        R, k = case["resp"], min(case["topk"], case["prefix"])
        keys = R * k + R * (R + 1) // 2
        rows = min(case["prefix"], R * k) + R       # each latent row once
        nbytes = rows * 1152 + R * k * 4 + R * 128 * (576 * 2 + 512 * 4 + 512 * 2 + 576 * 4 + 4)
        return {"bytes": nbytes, "flops": 2 * 128 * keys * ((576 + 512) + (576 + 512 + 576))}
    R, P, H = case["resp"], case["prefix"], case["heads"]
    return {"bytes": P * 256 + R * (P * 4 + H * 260 + 8 * case["topk"]),
            "flops": 2 * 128 * H * R * P}


def tolerance(case):
    if case["kind"] == "dsa":
        # 32-bit sums of exact products; the same scores give the same selection
        return {"rel": 1e-5, "max": 1e-4, "differ": 0.005}
    if case.get("dtype") == "f32":
        # dq of a row is what is left of terms P (dP - Delta) that cancel: up to
        # 2e-5 from the 64-bit value over a 32,000-position prefix
        return {"rel": 8e-5}
    if case["kind"] == "sparse":
        return {"rel": 4e-3, "max": 0.15}     # bf16 probabilities and dS; 1.1e-3 from 64 bits
    # bf16 probabilities, dS and outputs: 2e-3 to 4e-3 from 64 bits, dq up to 1e-2
    return {"rel": 7e-3 if case["kind"] == "capture" else 1e-2, "max": 0.3}


# ------------------------------------------------------------------ the same in 64 bits
def _rows64(pool, table, b, e, g):
    """Rows [b, e) of KV head g of a paged pool, as float64."""
    S = pool.shape[1]
    j = torch.arange(b, e, device=_DEV)
    return pool[table[j // S].long(), j % S, g].double()


def _attn64(q, k_of, v_of, hkv, q_pos0, kv_len, scale, d_out=None, prefix=0):
    """Causal attention of q [R, Hq, D] over kv_len positions; with d_out also
    dq and the dk, dv of positions >= prefix."""
    R, hq, D = q.shape
    G = hq // hkv
    Dv = v_of(0, 1, 0).shape[1]
    f64 = dict(dtype=torch.float64, device=_DEV)
    out, lse = torch.zeros((R, hq, Dv), **f64), torch.zeros((hq, R), **f64)
    dq = torch.zeros((R, hq, D), **f64)
    dk, dv = torch.zeros((kv_len - prefix, hkv, D), **f64), torch.zeros((kv_len - prefix, hkv, Dv),
                                                                      **f64)
    step = max(512, min(65_536, (1 << 27) // (R * G)))
    row_pos = (q_pos0 + torch.arange(R, device=_DEV)).repeat_interleave(G)[:, None]
    for g in range(hkv):
        qg = q[:, g * G:(g + 1) * G].double().reshape(R * G, D)

        def scores(b, e, k):
            s = (qg @ k.t()) * scale
            if e > q_pos0:
                s.masked_fill_(torch.arange(b, e, device=_DEV)[None, :] > row_pos, -math.inf)
            return s

        m = torch.full((R * G, 1), -math.inf, **f64)
        l, o = torch.zeros((R * G, 1), **f64), torch.zeros((R * G, Dv), **f64)
        for b in range(0, kv_len, step):
            e = min(kv_len, b + step)
            s = scores(b, e, k_of(b, e, g))
            m2 = torch.maximum(m, s.amax(1, keepdim=True))
            a = torch.exp(m - m2)
            p = s.sub_(m2).exp_()
            l = l * a + p.sum(1, keepdim=True)
            o = o * a + p @ v_of(b, e, g)
            m = m2
        o /= l
        L = m + l.log()
        out[:, g * G:(g + 1) * G] = o.view(R, G, Dv)
        lse[g * G:(g + 1) * G] = L.view(R, G).t()
        if d_out is None:
            continue
        dog = d_out[:, g * G:(g + 1) * G].double().reshape(R * G, Dv)
        delta = (dog * o).sum(1, keepdim=True)
        acc = torch.zeros((R * G, D), **f64)
        for b in range(0, kv_len, step):
            e = min(kv_len, b + step)
            k, v = k_of(b, e, g), v_of(b, e, g)
            p = scores(b, e, k).sub_(L).exp_()
            ds = (dog @ v.t()).sub_(delta).mul_(p)
            acc += ds @ k
            if e > prefix:
                x = max(b, prefix)
                dv[x - prefix:e - prefix, g] = p[:, x - b:].t() @ dog
                dk[x - prefix:e - prefix, g] = (ds[:, x - b:].t() @ qg) * scale
        dq[:, g * G:(g + 1) * G] = (acc * scale).view(R, G, D)
    return out, lse, dq, dk, dv


def exact(case, seed):
    kind = case["kind"]
    if work(case)["flops"] > 6e13:
        return None
    if kind == "replay":
        cfg, d = _replay_inputs(case, seed)
        out, lse, dq, dk, dv = _attn64(
            d["q"], lambda b, e, g: _rows64(d["k_pool"], d["page_table"], b, e, g),
            lambda b, e, g: _rows64(d["v_pool"], d["page_table"], b, e, g), cfg.n_kv_heads,
            cfg.q_pos0, cfg.kv_len, cfg.scale, d["d_out"] if case["bwd"] else None, cfg.prefix_len)
        r = dict(out=out, lse=lse)
        return dict(r, dq=dq, dk=dk, dv=dv) if case["bwd"] else r
    if kind == "blockwise":
        cfg, store, d = _blockwise_inputs(case, seed)
        P, table = cfg.prefix_len, store["prefix_table"]

        def rows(pool, own):
            return lambda b, e, g: torch.cat([_rows64(pool, table, min(b, P), min(e, P), g),
                                              own[max(b, P) - P:max(e, P) - P, g].double()])

        _, _, dq, dk, dv = _attn64(d["q"], rows(store["k_pool"], d["k"]),
                                   rows(store["v_pool"], d["v"]), 2, P, cfg.kv_len, cfg.scale,
                                   d["d_out"], P)
        return dict(dq=dq, dk=dk, dv=dv)
    if kind == "capture":
        cfg, d = _capture_inputs(case, seed)
        out = torch.empty((cfg.length, 16, 256), dtype=torch.float64, device=_DEV)
        for c in range(cfg.n_chunks):
            b, e = cfg.chunk_range(c)
            out[b:e] = _attn64(d["q_blocks"][c, :e - b], lambda x, y, g: d["k"][x:y, g].double(),
                               lambda x, y, g: d["v"][x:y, g].double(), 2, b, e, cfg.scale,
                               None, e)[0]
        pools = []
        for x in (d["k"], d["v"]):
            flat = torch.zeros((cfg.n_logical_pages * 256, 2, 256), dtype=torch.float64,
                               device=_DEV)
            flat[:cfg.length] = x.double()
            pool = torch.empty_like(flat).view(-1, 256, 2, 256)
            pool[d["page_table"].long()] = flat.view(-1, 256, 2, 256)
            pools.append(pool)
        return dict(out=out, k_pool=pools[0], v_pool=pools[1])
    if kind == "sparse":
        d = _sparse_inputs(case, seed)
        R, P, scale = case["resp"], case["prefix"], 576 ** -0.5
        f64 = dict(dtype=torch.float64, device=_DEV)
        out, lse = torch.empty((R, 128, 512), **f64), torch.empty((128, R), **f64)
        dq = torch.empty((R, 128, 576), **f64)
        flat = d["pool"].view(-1, 576)
        for t in range(R):
            pos = torch.cat([d["idx"][t].long(), torch.arange(P, P + t + 1, device=_DEV)])
            k = flat[d["table"][pos // 64].long() * 64 + pos % 64].double()
            v = k[:, :512].contiguous()
            s = (d["q"][t].double() @ k.t()) * scale
            lse[:, t] = torch.logsumexp(s, 1)
            p = torch.exp(s - lse[:, t, None])
            out[t] = p @ v
            do = d["d_out"][t].double()
            ds = p * (do @ v.t() - (do * out[t]).sum(1, keepdim=True))
            dq[t] = (ds @ k) * scale
        return dict(out=out, lse=lse, dq=dq)
    d = _dsa_inputs(case, seed)
    R, P, H = case["resp"], case["prefix"], case["heads"]
    scores = torch.empty((R, P), dtype=torch.float64, device=_DEV)
    flat = d["k_index_pool"].view(-1, 128)
    for b in range(0, P, 32_768):
        e = min(P, b + 32_768)
        j = torch.arange(b, e, device=_DEV)
        k = flat[d["page_table"][j // 64].long() * 64 + j % 64].double()
        for t0 in range(0, R, 64):
            t1 = min(R, t0 + 64)
            s = (d["q_index"][t0:t1].reshape(-1, 128).double() @ k.t()).clamp_(min=0)
            s = s.view(t1 - t0, H, e - b) * d["w_index"][t0:t1].double()[:, :, None]
            scores[t0:t1, b:e] = s.sum(1)
    return dict(idx=None, idx_scores=None, scores=scores)
