"""The binding's own workspaces belong to the stream that the call runs on, whatever form it is given in: torch gives the memory back to the
stream it was allocated under, and one allocated under another stream could be handed out again while the call's kernels are still queued."""
import contextlib

import numpy as np
import pytest
import torch

from paper_2603_22943_amd import taq as T


class Stream:
    """A stand-in for torch.cuda.Stream. As there, a handle of 0 counts as none: the stream is then a new one of torch's pool."""

    def __init__(self, handle):
        self.cuda_stream = handle or "pool"


class Handle:
    """A stream of another library: nothing but the raw handle."""

    def __init__(self, cuda_stream):
        self.cuda_stream = cuda_stream


DEFAULT, SIDE = Stream("default"), Stream(0x1234)
DEFAULT.cuda_stream = 0


@pytest.mark.parametrize("given,handle", [(None, "current"), (0, 0), (Handle(0), 0), (DEFAULT, 0), (SIDE, 0x1234), (0x1234, 0x1234), (Handle(0x1234), 0x1234)])
def test_scratch_is_allocated_under_the_given_stream(monkeypatch, given, handle):
    under = ["current"]

    @contextlib.contextmanager
    def stream(s):
        under.append(s.cuda_stream)
        yield
        under.pop()

    monkeypatch.setattr(torch.cuda, "Stream", Stream)
    monkeypatch.setattr(torch.cuda, "ExternalStream", lambda handle, device=None: Stream(handle))
    monkeypatch.setattr(torch.cuda, "default_stream", lambda device=None: DEFAULT)
    monkeypatch.setattr(torch.cuda, "stream", stream)
    monkeypatch.setattr(torch, "empty", lambda n, **_: under[-1])
    assert T._scratch(64, "cuda:0", given) == handle


@pytest.mark.gpu
@pytest.mark.parametrize("form", ["0", "default", "side", "side's handle"])
def test_calls_that_bring_their_own_workspace(monkeypatch, form):
    """On the GPU: the allocation's stream is the call's, and its results are those of a call with a workspace."""
    from test_gpu_token_tiles import Layer

    L = Layer(1, 100, 640, 8)
    want = L.run()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    given = {"0": 0, "default": torch.cuda.default_stream(), "side": side, "side's handle": side.cuda_stream}[form]
    s, out, under, empty = L.shape(L.N), torch.full_like(L.hidden, float("nan")), [], torch.empty
    torch.cuda.synchronize()

    def recorded(*args, **more):
        under.append(torch.cuda.current_stream().cuda_stream)
        return empty(*args, **more)

    monkeypatch.setattr(torch, "empty", recorded)
    with torch.cuda.stream(torch.cuda.Stream()):  # (the caller's current stream is another one)
        T.taq_cross_attn(L.hidden, L.kv, L.w, L.w, L.scales, L.mask, s, out, stream=given)
    monkeypatch.undo()
    torch.cuda.synchronize()
    assert under == [0 if form in ("0", "default") else side.cuda_stream]
    assert np.array_equal(out.cpu().numpy().view(np.uint16), want)
