"""Keys that no query of the call sees: their dK and dV are zero whatever their
rows hold, and the other keys' are the same, in every form of the pipelined
dK/dV kernel, with cut and with whole walks."""
import pytest
import torch

import paper_2609_19242_amd as bd
from paper_2609_19242_amd import CLEAN, CORRUPTED, Range

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("hilo", [0, bd.HILO_ALL | bd.HILO_ADAPTIVE], ids=["single", "adaptive"])
@pytest.mark.parametrize("Hq", [2, 3])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("rows,M", [(64, 16), (1600, 100)], ids=["whole", "cut"])
def test_unseen_keys(rows, M, D, Hq, hilo):
    L = rows + 4 * M
    g = torch.Generator().manual_seed(8)
    draw = lambda n, h: torch.randn(1, n, h, D, generator=g).to(torch.bfloat16).to(DEV)  # noqa: E731
    q, do, k, v = draw(rows, Hq), draw(rows, Hq), draw(L, 1), draw(L, 1)
    p = bd.make_problem(1, L, M, Hq, 1, D, torch.bfloat16, out_f32=True, hilo=hilo)
    QR, KR = [Range(CORRUPTED, 0, rows)], [Range(CLEAN, 0, L)]
    o, lse = torch.empty(1, rows, Hq, D, device=DEV), torch.empty(1, Hq, rows, device=DEV)
    bd.attn_fwd(p, QR, [q], [o], [lse], KR, [k], [v])
    seen = rows - M  # the clean context of the last block ends here
    ws = torch.empty(bd.attn_bwd_workspace_bytes(p, QR), dtype=torch.uint8, device=DEV)
    cut = ws.numel() > 2 * (-(-rows * Hq * 4 // 256) * 256)
    assert cut == (rows > 64)

    def grads(k, v):
        dk, dv = (torch.full((1, L, 1, D), 7.0, device=DEV) for _ in range(2))
        bd.attn_bwd(p, QR, [q], [o], [lse], [do], [torch.empty_like(o)], KR, [k], [v], [dk], [dv], ws)
        torch.cuda.synchronize()
        return dk, dv

    want = grads(k, v)
    kb, vb = k.clone(), v.clone()
    kb[:, seen] = float("nan")
    kb[:, seen + 3, :, ::2] = float("inf")
    kb[:, seen + 5] = float("-inf")
    vb[:, seen + 9] = float("nan")
    vb[:, seen + 5, :, ::3] = float("inf")
    for a, b in zip(grads(kb, vb), want):
        assert bool((a[:, seen:] == 0).all())
        assert torch.equal(a, b)
