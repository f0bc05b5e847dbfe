"""joint_bwd on a stream of the caller's choice with a workspace of its own: the
workspace is kept for that stream, in whichever form the stream is given."""
import pytest
import torch

import paper_2609_19242_amd as bd
from tests.gpu_util import joint_inputs

DEV = "cuda"


class _Handle:  # another wrapper of a raw stream, as other libraries pass it
    def __init__(self, handle):
        self.cuda_stream = handle


def test_default_stream_handle_is_the_default_stream(monkeypatch):
    monkeypatch.setattr(torch.cuda, "default_stream", lambda device: ("default", device))
    monkeypatch.setattr(torch.cuda, "ExternalStream", lambda handle, device: (handle, device))
    assert bd._torch_stream(0, "d") == ("default", "d")
    assert bd._torch_stream(_Handle(0), "d") == ("default", "d")
    assert bd._torch_stream(77, "d") == (77, "d")


@pytest.mark.gpu
@pytest.mark.parametrize("form", ["stream", "handle", "wrapper"])
@pytest.mark.parametrize("which", ["default", "side"])
def test_workspace_is_recorded_on_the_stream(which, form, monkeypatch):
    L, M, Hq, Hkv, D = 1024, 32, 4, 2, 128  # cut walks: the workspace holds partial sums
    q, k, v, do = (t.to(DEV) for t in joint_inputs(L, Hq, Hkv, D, torch.bfloat16, seed=3))
    o, lse = bd.joint_fwd(q, k, v, M)
    want = bd.joint_bwd(q, k, v, o, lse, do, M)
    st = torch.cuda.default_stream() if which == "default" else torch.cuda.Stream()
    other = torch.cuda.Stream()
    torch.cuda.synchronize()
    recorded = []
    keep = torch.Tensor.record_stream
    monkeypatch.setattr(torch.Tensor, "record_stream",
                        lambda t, s: (recorded.append((s.cuda_stream, s.device)), keep(t, s))[1])
    arg = {"stream": st, "handle": st.cuda_stream, "wrapper": _Handle(st.cuda_stream)}[form]
    with torch.cuda.stream(other):  # the caller's current stream, on which the workspace is allocated
        grads = tuple(torch.empty_like(t) for t in (q, k, v))
        for _ in range(4):
            bd.joint_bwd(q, k, v, o, lse, do, M, out=grads, stream=arg)
    torch.cuda.synchronize()
    assert recorded == [(st.cuda_stream, q.device)] * 4
    for a, b in zip(grads, want):
        assert torch.equal(a, b)
