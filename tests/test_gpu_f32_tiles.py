"""The fp32 kernels at the edges of their 16-row tiles, with and without cut
dK/dV walks, against the fp64 oracle (the fp32 bar, 1e-5), and the isolation of
hidden rows: an infinity or NaN in a row nobody sees changes nothing."""
import pytest
import torch

import oracle
import paper_2609_19242_amd as bd
from tests.gpu_util import assert_close, joint_inputs

pytestmark = pytest.mark.gpu
DEV = "cuda"

# L, block, heads, kv_heads, head_dim, batch, reading, window: two rows (dS of one key is 0), one tile and one more or less, several
# ranges' worth of tiles per wave, odd groups, a window inside a tile, walks long enough to be cut
SHAPES = [(2, 2, 1, 1, 64, 1, 0, 0), (15, 5, 3, 1, 128, 2, 1, 0), (17, 17, 2, 2, 64, 1, 0, 0),
          (33, 11, 4, 2, 128, 1, 1, 3), (129, 3, 2, 1, 64, 3, 0, 20), (500, 25, 4, 2, 128, 1, 0, 0),
          (272, 16, 6, 2, 64, 2, 1, 0)]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_fp32_tile_edges(shape):
    L, M, Hq, Hkv, D, B, reading, window = shape
    q, k, v, do = joint_inputs(L, Hq, Hkv, D, torch.float32, batch=B, seed=300 + L)
    O, LSE = oracle.joint_fwd(q, k, v, L, M, clean_intra=reading, window=window)
    ref = oracle.joint_bwd(q, k, v, O, LSE, do, L, M, clean_intra=reading, window=window)
    qd, kd, vd, dod = (t.to(DEV) for t in (q, k, v, do))
    o, lse = bd.joint_fwd(qd, kd, vd, M, reading, window=window)
    p = bd.make_problem(B, L, M, Hq, Hkv, D, torch.float32, clean_intra=reading, window=window)
    r = bd.joint_ranges(L)
    # room for the row statistics only (two fp32 arrays per range, rounded up to 256 bytes): whole walks
    whole = torch.empty(2 * 2 * (-(-B * L * Hq * 4 // 256) * 256), dtype=torch.uint8, device=DEV)
    cut = bd.attn_bwd_workspace_bytes(p, r)
    assert cut >= whole.numel()
    assert L < 500 or cut > whole.numel()  # the longest shape's walks are cut
    for ws in (whole, None):
        grads = bd.joint_bwd(qd, kd, vd, o, lse, dod, M, reading, window=window, workspace=ws)
        for name, got, want in zip(("O", "LSE", "dQ", "dK", "dV"), (o, lse) + grads, (O, LSE) + ref):
            assert_close(f"{shape} {'whole' if ws is not None else 'cut'} {name}", got, want, torch.float32)


@pytest.mark.parametrize("D", [64, 128])
def test_fp32_hidden_rows_stay_apart(D):
    L, M, Hq, Hkv, r = 48, 16, 2, 1, 20
    q, k, v, do = (t.to(DEV) for t in joint_inputs(L, Hq, Hkv, D, torch.float32, seed=77))
    o, lse = bd.joint_fwd(q, k, v, M)
    dq, dk, dv = bd.joint_bwd(q, k, v, o, lse, do, M)
    unseen = list(range(0, 32)) + list(range(L, L + r))  # query rows that do not see clean key r
    for bad in (float("inf"), float("nan")):
        kb, vb = k.clone(), v.clone()
        kb[:, L + r] = bad
        vb[:, L + r, :, ::3] = bad
        ob, lb = bd.joint_fwd(q, kb, vb, M)
        assert torch.equal(ob[:, unseen], o[:, unseen]) and torch.equal(lb[:, :, unseen], lse[:, :, unseen])
        dqb = bd.joint_bwd(q, kb, vb, o, lse, do, M)[0]
        assert torch.equal(dqb[:, unseen], dq[:, unseen])
        qb, dob = q.clone(), do.clone()
        qb[:, L + r] = bad
        dob[:, L + r, :, ::5] = bad
        later = slice(L + r + 1, 2 * L)  # clean keys that query row r does not see
        _, dkb, dvb = bd.joint_bwd(qb, k, v, o, lse, dob, M)
        assert torch.equal(dkb[:, later], dk[:, later]) and torch.equal(dvb[:, later], dv[:, later])
