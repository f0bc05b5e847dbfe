"""The workloads whose speed this repository is judged by, with their reference values.

A case is one pass of BDLM attention through the Python package, the way a training program calls it: the
forward followed by the backward of one attention layer (``joint``), the same for a DFlash2 drafter layer
(``drafter``), or one context-sharded rank's share: a partial forward per key range, their log-sum-exp merge
and the backward over all key ranges (``csbp``).  Each returns the attention output, its LSE and the three
gradients.
"""
import math

import torch

import paper_2609_19242_amd as bd

CLEAN, CORRUPTED = bd.CLEAN, bd.CORRUPTED


def _case(kind, name=None, **kw):
    c = dict(kind=kind, batch=1, L=0, block=0, heads=0, kv_heads=0, dim=128, dtype="bf16", window=0,
             block_reading=False, adaptive=False, draft_blocks=0, shards=0, rank=0)
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # Smallest call: the fp32 workload on which the method's exactness is checked; launch and latency count.
        _case("joint", "tiny_fp32", L=256, block=16, heads=2, kv_heads=2, dim=64, dtype="fp32"),
        # An fp32 layer of a small model (verification runs, fp32 fine-tuning), ragged in every tile.
        _case("joint", "ragged_fp32", L=1125, block=25, heads=8, kv_heads=2, dim=128, dtype="fp32"),
        # Smallest bf16 call: a short sequence of a small model, where launches and latency count.
        _case("joint", "small_256", L=256, block=16, heads=4, kv_heads=2),
        # A short-context layer that fills the card only just, with block and tile edges that do not meet.
        _case("joint", "short_2040", L=2040, block=24, heads=32, kv_heads=8),
        # The ordinary training size: 4K context, batch 2.
        _case("joint", "step_4k", batch=2, L=4096, block=32, heads=32, kv_heads=8),
        # The same size for models of head dimension 64.
        _case("joint", "step_4k_d64", batch=2, L=4096, block=32, heads=32, kv_heads=8, dim=64),
        # Multi-head attention without grouping (one query head per KV head), ragged length, block reading.
        _case("joint", "mha_3000", L=3000, block=50, heads=16, kv_heads=16, block_reading=True),
        # A sliding-window layer of a long-context model (width 1,024).
        _case("joint", "window_32k", L=32768, block=64, heads=32, kv_heads=8, window=1024),
        # The long-context training step the method is made for: 32K context.
        _case("joint", "step_32k", L=32768, block=64, heads=32, kv_heads=8),
        # Keys of large norm, whose products carry a second bf16 term where a probability is large; fp32 outputs.
        _case("joint", "amplified_8k", L=8192, block=128, heads=32, kv_heads=4, adaptive=True),
        # One of 16 context-sharded ranks at 64K context: 4,096 corrupted rows over their own keys and 16 shards.
        _case("csbp", "csbp_64k", L=65536, block=32, heads=32, kv_heads=8, shards=16, rank=8),
        # A drafter layer: 512 draft blocks of 16 rows over 8K target features.
        _case("drafter", "drafter_8k", L=8192, block=16, heads=32, kv_heads=8, draft_blocks=512),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges."""
    kind = rng.choice(["joint"] * 6 + ["fp32", "csbp", "drafter"])
    block = _log(rng, 4, 128)
    dim = rng.choice([64, 128, 128])
    heads, kv = rng.choice([(4, 2), (16, 16), (24, 8), (32, 8), (32, 4), (12, 2)])
    if kind == "fp32":
        L = block * max(1, _log(rng, 256, 1500) // block)
        h, k = rng.choice([(2, 2), (8, 2), (6, 2)])
        return _case("joint", L=L, block=block, heads=h, kv_heads=k, dim=dim, dtype="fp32",
                     window=rng.choice([0, 0, _log(rng, 32, 512)]))
    if kind == "csbp":
        shards = rng.choice([4, 8, 16])
        per = max(1, _log(rng, 512, 65536 // 16) // block)
        return _case("csbp", L=block * per * shards, block=block, heads=heads, kv_heads=kv, dim=dim, shards=shards,
                     rank=rng.randrange(shards))
    if kind == "drafter":
        L = block * max(2, _log(rng, 1024, 16384) // block)
        return _case("drafter", L=L, block=block, heads=heads, kv_heads=kv, dim=dim,
                     draft_blocks=rng.randint(max(1, L // block // 8), L // block))
    L = block * max(2, _log(rng, 256, 16384) // block)
    batch = rng.choice([1, 1, 2, 3]) if L <= 4096 else 1
    opt = rng.choice(["", "", "window", "adaptive", "block_reading"])
    return _case("joint", batch=batch, L=L, block=block, heads=heads, kv_heads=kv, dim=dim,
                 window=_log(rng, 64, 2048) if opt == "window" else 0, adaptive=opt == "adaptive",
                 block_reading=opt == "block_reading")


# ------------------------------------------------------------------ rows of a case
def _q_ranges(c):
    """(stream, first position, rows) of the query rows, in order."""
    if c["kind"] == "joint":
        return [(CORRUPTED, 0, c["L"]), (CLEAN, 0, c["L"])]
    if c["kind"] == "drafter":
        return [(CORRUPTED, 0, c["draft_blocks"] * c["block"])]
    n = c["L"] // c["shards"]
    return [(CORRUPTED, c["rank"] * n, n)]


def _k_ranges(c):
    if c["kind"] == "joint":
        return [(CORRUPTED, 0, c["L"]), (CLEAN, 0, c["L"])]
    if c["kind"] == "drafter":
        return [(CORRUPTED, 0, c["draft_blocks"] * c["block"]), (CLEAN, 0, c["L"])]
    n = c["L"] // c["shards"]
    return [(CORRUPTED, c["rank"] * n, n)] + [(CLEAN, s * n, n) for s in range(c["shards"])]


def _rows(ranges, device):
    st = torch.cat([torch.full((n,), s, dtype=torch.int64, device=device) for s, _, n in ranges])
    pos = torch.cat([torch.arange(p, p + n, dtype=torch.int64, device=device) for _, p, n in ranges])
    return st, pos


def _anchor_table(c, seed, device):
    """Sorted anchors of the draft blocks; entries past the draft blocks end at L."""
    g = torch.Generator().manual_seed(1000003 * seed + 4)
    a = torch.sort(torch.randint(1, c["L"] + 1, (c["draft_blocks"],), generator=g)).values
    rest = torch.full((c["L"] // c["block"] - c["draft_blocks"],), c["L"])
    return torch.cat([a, rest]).to(torch.int32).to(device)


def _visible_bounds(c, table, st, pos):
    """Per query row: the visible clean keys [lo, hi) and corrupted keys [lo, hi) by position."""
    M = c["block"]
    blk = pos // M
    own = (blk + 1) * M if c["block_reading"] else pos + 1
    ctx = table.to(torch.int64)[blk] if table is not None else blk * M
    chi = torch.where(st == CLEAN, own, ctx)
    clo = torch.clamp(chi - c["window"], min=0) if c["window"] else torch.zeros_like(chi)
    corr = st == CORRUPTED
    zero = torch.zeros_like(pos)
    return clo, chi, torch.where(corr, blk * M, zero), torch.where(corr, (blk + 1) * M, zero)


def _pairs(c):
    """Visible query-key pairs per query head and batch element (a drafter's with evenly spread anchors)."""
    st, pos = _rows(_q_ranges(c), "cpu")
    table = None
    if c["kind"] == "drafter":
        n = c["draft_blocks"]
        table = torch.cat([(torch.arange(1, n + 1) * c["L"]) // (n + 1), torch.full((c["L"] // c["block"] - n,), c["L"])])
    clo, chi, blo, bhi = _visible_bounds(c, table, st, pos)
    tot = 0
    for s, p, n in _k_ranges(c):
        lo, hi = (clo, chi) if s == CLEAN else (blo, bhi)
        tot += int((torch.clamp(hi, max=p + n) - torch.clamp(lo, min=p)).clamp(min=0).sum())
    return tot


# ------------------------------------------------------------------ the pass
def _normal(shape, seed, t, dtype, device="cuda"):
    g = torch.Generator(device=device).manual_seed(1000003 * seed + t)
    return torch.randn(*shape, generator=g, dtype=torch.float32, device=device).to(dtype)


def prepare(case, seed):
    """Projections Q, K, V of unit variance and the upstream gradient, as a layer holds them before the call."""
    c = case
    dt = torch.float32 if c["dtype"] == "fp32" else torch.bfloat16
    nq = sum(n for _, _, n in _q_ranges(c))
    nk = sum(n for _, _, n in _k_ranges(c))
    H, KV, D = c["heads"], c["kv_heads"], c["dim"]
    s = dict(case=c, q=_normal((c["batch"], nq, H, D), seed, 0, dt), v=_normal((c["batch"], nk, KV, D), seed, 2, dt),
             do=_normal((c["batch"], nq, H, D), seed, 3, dt), table=None)
    k = _normal((c["batch"], nk, KV, D), seed, 1, torch.float32)
    if c["adaptive"]:  # 1% of the keys eight times as long
        g = torch.Generator().manual_seed(1000003 * seed + 5)
        idx = torch.randperm(nk, generator=g)[:max(1, nk // 100)].to("cuda")
        k[:, idx] *= 8
    s["k"] = k.to(dt)
    if c["kind"] == "drafter":
        s["table"] = _anchor_table(c, seed, "cuda")
    if c["kind"] != "joint":
        s["problem"] = bd.make_problem(1, c["L"], c["block"], H, KV, D, dt, clean_prefix=s["table"])
        s["qr"] = [bd.Range(*r) for r in _q_ranges(c)]
        s["kr"] = [bd.Range(*r) for r in _k_ranges(c)]
        sizes = [r[2] for r in _k_ranges(c)]
        s["ks"], s["vs"] = list(s["k"].split(sizes, 1)), list(s["v"].split(sizes, 1))
        s["workspace"] = torch.empty(bd.attn_bwd_workspace_bytes(s["problem"], s["qr"]), dtype=torch.uint8,
                                     device="cuda")
    if c["kind"] == "csbp":  # buffers a rank keeps for its partials
        s["parts"] = [torch.empty_like(s["q"]) for _ in s["kr"]]
        s["part_lse"] = [torch.empty(1, H, nq, device="cuda") for _ in s["kr"]]
    return s


def run(state):
    s = state
    c = s["case"]
    if c["kind"] == "joint":
        kw = dict(window=c["window"], out_f32=c["adaptive"],
                  clean_intra=bd.CLEAN_INTRA_BLOCK if c["block_reading"] else bd.CLEAN_INTRA_CAUSAL,
                  hilo=bd.HILO_ALL | bd.HILO_ADAPTIVE if c["adaptive"] else False)
        o, lse = bd.joint_fwd(s["q"], s["k"], s["v"], c["block"], **kw)
        dq, dk, dv = bd.joint_bwd(s["q"], s["k"], s["v"], o, lse, s["do"], c["block"], **kw)
        return o, lse, dq, dk, dv
    p, qr, kr, ks, vs = s["problem"], s["qr"], s["kr"], s["ks"], s["vs"]
    o = torch.empty_like(s["q"])
    lse = torch.empty(1, c["heads"], s["q"].shape[1], device="cuda")
    if c["kind"] == "drafter":
        bd.attn_fwd(p, qr, [s["q"]], [o], [lse], kr, ks, vs)
    else:
        for j in range(len(kr)):
            bd.attn_partial_fwd(p, qr[0], s["q"], s["parts"][j], s["part_lse"][j], kr[j], ks[j], vs[j])
        bd.lse_merge(s["parts"], s["part_lse"], o, lse)
    dq, dk, dv = torch.empty_like(s["q"]), torch.empty_like(s["k"]), torch.empty_like(s["v"])
    sizes = [r.len for r in kr]
    bd.attn_bwd(p, qr, [s["q"]], [o], [lse], [s["do"]], [dq], kr, ks, vs, list(dk.split(sizes, 1)),
                list(dv.split(sizes, 1)), s["workspace"])
    return o, lse, dq, dk, dv


def work(case):
    """Inputs and outputs once; 4 d operations per visible pair forward and 10 d backward."""
    c = case
    e = 4 if c["dtype"] == "fp32" else 2
    eo = 4 if c["adaptive"] else e
    nq = sum(n for _, _, n in _q_ranges(c)) * c["batch"] * c["heads"]
    nk = sum(n for _, _, n in _k_ranges(c)) * c["batch"] * c["kv_heads"]
    d = c["dim"]
    return {"bytes": d * (2 * nq + 2 * nk) * e + d * (2 * nq + 2 * nk) * eo + 4 * nq,
            "flops": 14 * d * _pairs(c) * c["heads"] * c["batch"]}


def tolerance(case):
    """About four times the measured distance from 64-bit arithmetic: 1.3e-7 in fp32 (sums in 64 bits, LSE and
    results rounded to 32), 2.1e-4 with fp32 outputs and two-term products, 2.9e-3 with bf16 outputs."""
    if case["dtype"] == "fp32":
        return {"rel": 5e-7}
    return {"rel": 1e-3 if case["adaptive"] else 1e-2}


# ------------------------------------------------------------------ 64-bit values
def exact(case, seed):
    c = case
    if _pairs(c) * c["heads"] * c["batch"] > 6e10:
        return None
    s = prepare(c, seed)
    st, pos = _rows(_q_ranges(c), "cuda")
    ks, kp = _rows(_k_ranges(c), "cuda")
    clo, chi, blo, bhi = _visible_bounds(c, s["table"], st, pos)
    B, nq, H, D = s["q"].shape
    nk, KV = s["k"].shape[1:3]
    scale = 1.0 / math.sqrt(D)
    f64 = dict(dtype=torch.float64, device="cuda")
    o, dq = torch.empty(B, nq, H, D, **f64), torch.empty(B, nq, H, D, **f64)
    lse = torch.empty(B, H, nq, **f64)
    dk, dv = torch.zeros(B, nk, KV, D, **f64), torch.zeros(B, nk, KV, D, **f64)
    chunk = 2048
    for r0 in range(0, nq, chunk):
        r = slice(r0, min(nq, r0 + chunk))
        vis = torch.where((ks == CLEAN)[None], (kp[None] >= clo[r, None]) & (kp[None] < chi[r, None]),
                          (kp[None] >= blo[r, None]) & (kp[None] < bhi[r, None]))
        cols = torch.nonzero(vis.any(0)).flatten()  # keys some row of the chunk sees
        vis = ~vis[:, cols]
        for b in range(B):
            for h in range(H):
                g = h // (H // KV)
                q, do = s["q"][b, r, h].double(), s["do"][b, r, h].double()
                k, v = s["k"][b, cols, g].double(), s["v"][b, cols, g].double()
                sc = torch.mm(q, k.t().contiguous()).mul_(scale).masked_fill_(vis, -math.inf)
                z = torch.logsumexp(sc, 1)
                p = sc.sub_(z[:, None]).exp_()
                oo = torch.mm(p, v)
                o[b, r, h], lse[b, h, r] = oo, z
                dv[b, :, g].index_add_(0, cols, torch.mm(p.t().contiguous(), do))
                ds = torch.mm(do, v.t().contiguous()).sub_((do * oo).sum(1, keepdim=True)).mul_(p)
                dq[b, r, h] = torch.mm(ds, k) * scale
                dk[b, :, g].index_add_(0, cols, torch.mm(ds.t().contiguous(), q) * scale)
    return o, lse, dq, dk, dv
