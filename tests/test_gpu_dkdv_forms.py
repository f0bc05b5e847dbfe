"""The forms of the pipelined dK/dV kernel against the fp64 oracle: head_dim 64
and 128, steps of two heads (even GQA groups) and of 64 rows of one head (odd
ones), single-term and adaptive two-term products, at the edges of its 32- and
64-row blocks and 128-key tiles, and two query ranges in either order with
spans apart.  fp32 outputs, the bf16 bar."""
import pytest
import torch

import oracle
import paper_2609_19242_amd as bd
from paper_2609_19242_amd import CLEAN, CORRUPTED, Range
from tests.gpu_util import assert_close, joint_inputs

pytestmark = pytest.mark.gpu
DEV = "cuda"
ADAPT = bd.HILO_ALL | bd.HILO_ADAPTIVE

SHAPES = [(63, 9, 3, 1, 1, 0, 0), (64, 16, 1, 1, 2, 1, 0), (65, 13, 5, 5, 1, 0, 0), (129, 43, 3, 3, 1, 1, 30),
          (260, 20, 2, 1, 2, 0, 0), (512, 64, 6, 2, 1, 0, 100)]  # L, block, heads, kv_heads, batch, reading, window


@pytest.mark.parametrize("hilo", [0, ADAPT], ids=["single", "adaptive"])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_dkdv_forms(shape, D, hilo):
    L, M, Hq, Hkv, B, reading, window = shape
    q, k, v, do = joint_inputs(L, Hq, Hkv, D, torch.bfloat16, batch=B, seed=700 + L)
    mask = dict(clean_intra=reading, window=window)
    O, LSE = oracle.joint_fwd(q, k, v, L, M, **mask)
    _, dK, dV = oracle.joint_bwd(q, k, v, O, LSE, do, L, M, **mask)
    qd, kd, vd, dod = (t.to(DEV) for t in (q, k, v, do))
    o, lse = bd.joint_fwd(qd, kd, vd, M, reading, out_f32=True, hilo=hilo, window=window)
    _, dk, dv = bd.joint_bwd(qd, kd, vd, o, lse, dod, M, reading, out_f32=True, hilo=hilo, window=window)
    assert_close(f"{shape} d{D} dK", dk, dK, torch.bfloat16)
    assert_close(f"{shape} d{D} dV", dv, dV, torch.bfloat16)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("spans", [((CLEAN, 200, 150), (CORRUPTED, 0, 70)), ((CORRUPTED, 300, 100), (CLEAN, 10, 95))])
def test_two_ranges_apart_odd_group(spans, D):
    L, M, Hq, Hkv = 400, 20, 3, 1
    q, k, v, do = joint_inputs(L, Hq, Hkv, D, torch.bfloat16, seed=44)
    rows = lambda t: [t[:, (L if s == CLEAN else 0) + p:(L if s == CLEAN else 0) + p + n].contiguous()  # noqa: E731
                      for s, p, n in spans]
    kspec = [(CORRUPTED, 0, L), (CLEAN, 0, L)]
    qs, dos = rows(q), rows(do)
    O, LSE = oracle.fwd(torch.cat(qs, 1), k, v, list(spans), kspec, M)
    dQ, dK, dV = oracle.bwd(torch.cat(qs, 1), k, v, O, LSE, torch.cat(dos, 1), list(spans), kspec, M)
    p = bd.make_problem(1, L, M, Hq, Hkv, D, torch.bfloat16, out_f32=True)
    QR, KR = [Range(*s) for s in spans], [Range(*s) for s in kspec]
    qd, dod = [t.to(DEV) for t in qs], [t.to(DEV) for t in dos]
    ks, vs = ([t[:, :L].contiguous().to(DEV), t[:, L:].contiguous().to(DEV)] for t in (k, v))
    o = [torch.empty(t.shape, device=DEV) for t in qd]
    lse = [torch.empty((1, Hq, t.shape[1]), device=DEV) for t in qd]
    bd.attn_fwd(p, QR, qd, o, lse, KR, ks, vs)
    dq = [torch.empty(t.shape, device=DEV) for t in qd]
    dk, dv = [torch.empty(t.shape, device=DEV) for t in ks], [torch.empty(t.shape, device=DEV) for t in ks]
    ws = torch.empty(bd.attn_bwd_workspace_bytes(p, QR), dtype=torch.uint8, device=DEV)
    bd.attn_bwd(p, QR, qd, o, lse, dod, dq, KR, ks, vs, dk, dv, ws)
    torch.cuda.synchronize()
    assert_close("dQ", torch.cat(dq, 1), dQ, torch.bfloat16)
    assert_close("dK", torch.cat(dk, 1), dK, torch.bfloat16)
    assert_close("dV", torch.cat(dv, 1), dV, torch.bfloat16)
