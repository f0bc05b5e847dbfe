"""The forward with two teams per workgroup (calls of at most 256 128-row query
tiles) against the fp64 oracle: one key tile and several (team 1 idle, odd and
even tile counts), ragged rows, rows that see no key, several key ranges, both
head dims and all three forms of P; and the one-team form at the other side of
the limit."""
import os
import re

import pytest
import torch

import oracle
import paper_2609_19242_amd as bd
from paper_2609_19242_amd import CLEAN, CORRUPTED, Range
from tests.gpu_util import assert_close, joint_inputs

DEV = "cuda"

# L, block, heads, kv_heads, batch, window
SHAPES = [(32, 8, 2, 1, 1, 0), (70, 10, 4, 2, 2, 0), (200, 25, 2, 2, 1, 30), (513, 27, 2, 1, 1, 0),
          (1024, 64, 16, 2, 1, 0), (258, 3, 43, 1, 1, 0), (129, 3, 43, 1, 2, 0)]
CSRC = os.path.join(os.path.dirname(os.path.abspath(bd.__file__)), "csrc")


def query_tiles(shape):
    """128-row query tiles of the call: two ranges of L rows."""
    L, _, Hq, _, B, _ = shape
    return 2 * -(-L // 128) * Hq * B


def test_shapes_reach_both_sides_of_the_limit():
    limit = int(re.search(r"kTeamWgs = (\d+);", open(os.path.join(CSRC, "common.hpp")).read()).group(1))
    tiles = [query_tiles(s) for s in SHAPES]
    assert limit == 256 and max(t for t in tiles if t <= limit) == limit, tiles
    assert min(t for t in tiles if t > limit) == limit + 2, tiles  # two equal ranges: an even count


@pytest.mark.gpu
@pytest.mark.parametrize("hilo", [0, bd.HILO_ALL, bd.HILO_ALL | bd.HILO_ADAPTIVE], ids=["single", "two", "adaptive"])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_forward_teams(shape, D, hilo):
    L, M, Hq, Hkv, B, window = shape
    q, k, v, _ = joint_inputs(L, Hq, Hkv, D, torch.bfloat16, batch=B, seed=900 + L)
    heads = [0, Hq - 1]
    O, LSE = oracle.joint_fwd(q, k, v, L, M, heads=heads, window=window)
    o, lse = bd.joint_fwd(q.to(DEV), k.to(DEV), v.to(DEV), M, out_f32=True, hilo=hilo, window=window)
    assert_close(f"{shape} d{D} O", o[:, :, heads], O, torch.bfloat16)
    assert_close(f"{shape} d{D} LSE", lse[:, heads], LSE, torch.bfloat16)


@pytest.mark.gpu
@pytest.mark.parametrize("D", [64, 128])
def test_partials_with_empty_rows(D):
    """Clean shards of 90 keys: rows of the first blocks see none of the later ones (O = 0, LSE = -inf), and
    the fused call over all of them runs over range changes inside a round."""
    L, M, H = 360, 12, 2
    q, k, v, _ = joint_inputs(L, H, 1, D, torch.bfloat16, seed=17)
    qc = q[:, :L].contiguous()
    spec = [(CLEAN, s, 90) for s in range(0, L, 90)] + [(CORRUPTED, 0, L)]
    part = lambda t, s, p, n: t[:, (L if s == CLEAN else 0) + p:(L if s == CLEAN else 0) + p + n].contiguous()  # noqa: E731
    p = bd.make_problem(1, L, M, H, 1, D, torch.bfloat16, out_f32=True)
    ks, vs = [part(k, *s) for s in spec], [part(v, *s) for s in spec]
    rows = [(CORRUPTED, 0, L)]
    for sel in ([0], [3], [4], [0, 1, 2, 3, 4]):
        sub = [spec[i] for i in sel]
        O, LSE = oracle.fwd(qc, torch.cat([ks[i] for i in sel], 1), torch.cat([vs[i] for i in sel], 1), rows, sub, M)
        o = torch.full((1, L, H, D), float("nan"), device=DEV)
        lse = torch.full((1, H, L), float("nan"), device=DEV)
        bd.attn_fwd(p, [Range(*rows[0])], [qc.to(DEV)], [o], [lse], [Range(*s) for s in sub],
                    [ks[i].to(DEV) for i in sel], [vs[i].to(DEV) for i in sel])
        torch.cuda.synchronize()
        assert_close(f"d{D} {sel} O", o, O, torch.bfloat16)
        assert_close(f"d{D} {sel} LSE", lse, LSE, torch.bfloat16)
