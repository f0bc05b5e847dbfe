"""dK/dV walks cut into chunks on calls small enough to be cut: against the fp64
oracle, and against the whole walk (a workspace with room for the row
statistics only), from which only the order of the fp32 sums differs (at most
some hundred terms are regrouped, so far below 1e-5 relative)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_19242_amd as bd
from paper_2609_19242_amd import CLEAN, CORRUPTED, Range
from tests.gpu_util import assert_close, joint_inputs

pytestmark = pytest.mark.gpu
DEV = "cuda"

# L, block, heads, kv_heads, batch, options; head_dim 128
CASES = [(1024, 32, 4, 2, 1, {}), (1100, 20, 2, 1, 1, {"clean_intra": 1}), (777, 21, 8, 2, 2, {}),
         (1024, 32, 4, 1, 1, {"hilo": bd.HILO_ALL | bd.HILO_ADAPTIVE}), (1536, 64, 4, 2, 1, {"window": 700})]


def stats_bytes(p, ranges):
    """The row statistics' part of the workspace: two fp32 arrays per query range, rounded up to 256 bytes."""
    return sum(2 * (-(-p.batch * r.len * p.heads * 4 // 256) * 256) for r in ranges)


def rel(a, b):
    return float((a.double() - b.double()).norm() / b.double().norm())


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"L{c[0]}-M{c[1]}-{c[2]}/{c[3]}-b{c[4]}-{'-'.join(c[5])}")
def test_cut_walks_joint(case):
    L, M, Hq, Hkv, B, opt = case
    q, k, v, do = joint_inputs(L, Hq, Hkv, 128, torch.bfloat16, batch=B, seed=500 + L)
    mask = {x: opt[x] for x in ("clean_intra", "window") if x in opt}
    O, LSE = oracle.joint_fwd(q, k, v, L, M, **mask)
    ref = oracle.joint_bwd(q, k, v, O, LSE, do, L, M, **mask)
    qd, kd, vd, dod = (t.to(DEV) for t in (q, k, v, do))
    r = bd.joint_ranges(L)
    for out_f32 in (True, False):
        p = bd.make_problem(B, L, M, Hq, Hkv, 128, torch.bfloat16, out_f32=out_f32, **opt)
        whole = torch.empty(stats_bytes(p, r), dtype=torch.uint8, device=DEV)
        assert bd.attn_bwd_workspace_bytes(p, r) > whole.numel()
        o, lse = bd.joint_fwd(qd, kd, vd, M, out_f32=out_f32, **opt)
        cut = bd.joint_bwd(qd, kd, vd, o, lse, dod, M, out_f32=out_f32, **opt)
        one = bd.joint_bwd(qd, kd, vd, o, lse, dod, M, out_f32=out_f32, workspace=whole, **opt)
        again = bd.joint_bwd(qd, kd, vd, o, lse, dod, M, out_f32=out_f32, **opt)
        torch.cuda.synchronize()
        for name, a, b, c, want in zip(("dQ", "dK", "dV"), cut, one, again, ref):
            assert torch.equal(a, c), name  # reproducible
            if out_f32:
                assert_close(f"{case} {name}", a, want, torch.bfloat16)
                assert rel(a, b) <= 1e-5, (name, rel(a, b))
            else:  # another order may move a sum across a bf16 rounding boundary
                assert rel(a, b) <= 2.0 ** -9, (name, rel(a, b))


@pytest.mark.parametrize("Hq", [2, 4])
def test_cut_walks_many_key_ranges(Hq):
    """A rank's share: one query range, its own corrupted keys and shards of the clean prefix, some ranges cut
    and some not, ragged tiles, an empty range, batch strides longer than the ranges."""
    L, M, Hkv, D = 3600, 30, 1, 128
    QR = [Range(CORRUPTED, 900, 1800, 1850)]
    spec = [(CORRUPTED, 900, 1800), (CLEAN, 0, 450), (CLEAN, 450, 0), (CLEAN, 450, 333), (CLEAN, 783, 1900)]
    KR = [Range(s, p, n, n + 7) for s, p, n in spec]
    g = torch.Generator().manual_seed(9)
    draw = lambda *sh: torch.randn(*sh, generator=g).to(torch.bfloat16)  # noqa: E731
    q, do = draw(2, 1850, Hq, D), draw(2, 1850, Hq, D)
    ks, vs = [draw(2, n + 7, Hkv, D) for _, _, n in spec], [draw(2, n + 7, Hkv, D) for _, _, n in spec]
    rows = [(CORRUPTED, 900, 1800)]
    kcat = torch.cat([k[:, :n] for k, (_, _, n) in zip(ks, spec)], 1)
    vcat = torch.cat([v[:, :n] for v, (_, _, n) in zip(vs, spec)], 1)
    O, LSE = oracle.fwd(q[:, :1800], kcat, vcat, rows, spec, M)
    dQ, dK, dV = oracle.bwd(q[:, :1800], kcat, vcat, O, LSE, do[:, :1800], rows, spec, M)
    p = bd.make_problem(2, L, M, Hq, Hkv, D, torch.bfloat16, out_f32=True)
    qd, dod, kd, vd = q.to(DEV), do.to(DEV), [t.to(DEV) for t in ks], [t.to(DEV) for t in vs]
    o = torch.full((2, 1850, Hq, D), float("nan"), device=DEV)
    lse = torch.full((2, Hq, 1850), float("nan"), device=DEV)
    bd.attn_fwd(p, QR, [qd], [o], [lse], KR, kd, vd)
    dq = torch.full_like(o, 7.0)
    dk, dv = [torch.full(t.shape, 7.0, device=DEV) for t in kd], [torch.full(t.shape, 7.0, device=DEV) for t in vd]
    n = bd.attn_bwd_workspace_bytes(p, QR)
    assert n > stats_bytes(p, QR)
    ws = torch.full((n + 4096,), 0xA5, dtype=torch.uint8, device=DEV)
    bd.attn_bwd(p, QR, [qd], [o], [lse], [dod], [dq], KR, kd, vd, dk, dv, ws[:n])
    torch.cuda.synchronize()
    assert bool((ws[n:] == 0xA5).all()), "written past the workspace"
    assert_close("dQ", dq[:, :1800], dQ, torch.bfloat16)
    at = 0
    for j, (_, _, len_) in enumerate(spec):
        if len_ == 0:
            continue
        assert_close(f"dK {j}", dk[j][:, :len_], dK[:, at:at + len_], torch.bfloat16)
        assert_close(f"dV {j}", dv[j][:, :len_], dV[:, at:at + len_], torch.bfloat16)
        assert bool((dk[j][:, len_:] == 7.0).all()) and bool((dv[j][:, len_:] == 7.0).all())
        at += len_
    assert np.isfinite(dQ).all()


@pytest.mark.parametrize("case", [(2660, 20, 56, 8, 128, 7, 6), (2112, 16, 16, 16, 64, 4, 3)],
                         ids=["380-row", "528-row"])
def test_cut_walks_do_not_depend_on_the_sharding(case):
    """A rank's backward over ragged shards of the clean keys and over the same keys as one range: the same chunks,
    so the same bits."""
    L, M, Hq, Hkv, D, shards, rank = case
    n = L // shards
    g = torch.Generator().manual_seed(21)
    draw = lambda rows, h: torch.randn(1, rows, h, D, generator=g).to(torch.bfloat16).to(DEV)  # noqa: E731
    q, do, k, v = draw(n, Hq), draw(n, Hq), draw(n + L, Hkv), draw(n + L, Hkv)
    QR = [Range(CORRUPTED, rank * n, n)]
    p = bd.make_problem(1, L, M, Hq, Hkv, D, torch.bfloat16, out_f32=True)
    ws = torch.empty(bd.attn_bwd_workspace_bytes(p, QR), dtype=torch.uint8, device=DEV)
    assert ws.numel() > stats_bytes(p, QR)
    o, lse = torch.empty(1, n, Hq, D, device=DEV), torch.empty(1, Hq, n, device=DEV)
    own = Range(CORRUPTED, rank * n, n)
    whole, parts = [own, Range(CLEAN, 0, L)], [own] + [Range(CLEAN, s * n, n) for s in range(shards)]
    got = []
    for kr in (whole, parts):
        sizes = [r.len for r in kr]
        split = lambda t: list(t.split(sizes, 1))  # noqa: B023, E731
        if kr is whole:
            bd.attn_fwd(p, QR, [q], [o], [lse], kr, split(k), split(v))
        dq = torch.empty_like(o)
        dk, dv = (torch.full((1, n + L, Hkv, D), 7.0, device=DEV) for _ in range(2))
        bd.attn_bwd(p, QR, [q], [o], [lse], [do], [dq], kr, split(k), split(v), split(dk), split(dv), ws)
        torch.cuda.synchronize()
        got.append((dk, dv))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    dk, dv = torch.empty_like(got[0][0]), torch.empty_like(got[0][1])
    small = torch.empty(stats_bytes(p, QR), dtype=torch.uint8, device=DEV)
    sizes = [r.len for r in whole]
    bd.attn_bwd(p, QR, [q], [o], [lse], [do], [torch.empty_like(o)], whole, list(k.split(sizes, 1)),
                list(v.split(sizes, 1)), list(dk.split(sizes, 1)), list(dv.split(sizes, 1)), small)
    torch.cuda.synchronize()
    assert rel(got[0][0], dk) <= 1e-5 and rel(got[0][1], dv) <= 1e-5  # whole walks


def test_noalloc_cuts_like_the_workspace_call():
    """Partial sums that would fill more than the scratch array at the average load per chunk."""
    L, M, H, D, B = 1080, 9, 16, 128, 2
    q, k, v, do = (t.to(DEV) for t in joint_inputs(L, H, H, D, torch.bfloat16, batch=B, seed=31))
    r = bd.joint_ranges(L)
    p = bd.make_problem(B, L, M, H, H, D, torch.bfloat16)
    assert stats_bytes(p, r) < bd.attn_bwd_workspace_bytes(p, r) <= bd.NOALLOC_SCRATCH_BYTES
    o, lse = bd.joint_fwd(q, k, v, M)
    want = bd.joint_bwd(q, k, v, o, lse, do, M)
    got = tuple(torch.empty_like(t) for t in (q, k, v))
    halves = lambda t: bd._joint_ptrs(t, L)  # noqa: E731
    dq, dk, dv = got
    bd.attn_bwd_noalloc(p, r, halves(q), halves(o), [lse.data_ptr(), lse.data_ptr() + L * 4], halves(do), halves(dq),
                        r, halves(k), halves(v), halves(dk), halves(dv))
    torch.cuda.synchronize()
    for name, a, b in zip(("dQ", "dK", "dV"), got, want):
        assert torch.equal(a, b), name
