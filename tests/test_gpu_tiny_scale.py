"""Softmax scales so small that LSE / scale passes the fp32 range (attention
close to uniform) in the backward, against the fp64 oracle: every form of the
dK/dV products, even and odd GQA groups, and the smallest scale of the
pipelined kernel beside it."""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_19242_amd as bd
from tests.gpu_util import assert_close, joint_inputs

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("hilo", [0, bd.HILO_ALL, bd.HILO_ALL | bd.HILO_ADAPTIVE], ids=["single", "two", "adaptive"])
@pytest.mark.parametrize("Hq", [2, 3])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("scale", [2.0 ** -127, 2.0 ** -97, 2.0 ** -96])
def test_tiny_scale(scale, D, Hq, hilo):
    L, M = 144, 16
    q, k, v, do = joint_inputs(L, Hq, 1, D, torch.bfloat16, seed=41)
    O, LSE = oracle.joint_fwd(q, k, v, L, M, scale=scale)
    dQ, dK, dV = oracle.joint_bwd(q, k, v, O, LSE, do, L, M, scale=scale)
    qd, kd, vd, dod = (t.to(DEV) for t in (q, k, v, do))
    o, lse = bd.joint_fwd(qd, kd, vd, M, scale=scale, out_f32=True, hilo=hilo)
    dq, dk, dv = bd.joint_bwd(qd, kd, vd, o, lse, dod, M, scale=scale, out_f32=True, hilo=hilo)
    assert_close(f"scale {scale} d{D} dV", dv, dV, torch.bfloat16)
    for name, got, want in (("dQ", dq, dQ), ("dK", dk, dK)):  # about 1e-29 and below, next to their bf16 bar
        if scale > 2.0 ** -120:  # (below, dK and dQ are subnormal)
            g = got.double().cpu().numpy()
            assert np.linalg.norm(g - want) <= 5e-3 * np.linalg.norm(want), name
