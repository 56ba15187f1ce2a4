"""The workspaces of SparseLinear: a buffer whose address a captured graph holds lives as long as the module
and serves no other call, and calls on different streams never share one. The rules on the CPU with a
stand-in for the encoded matrix; the replay of a graph after the module has moved on to a larger workspace on
the GPU."""
import gc
import types
import weakref

import numpy as np
import pytest
import torch

from paper_2607_08786_amd import linear, usp


class _Matrix:
    """Needs 100 bytes a token, none at one token."""

    def __init__(self, W, mask, device=0):
        pass

    def workspace_size(self, N):
        return 0 if N == 1 else 100 * N

    def make_workspace(self, N, stream=None):
        return torch.zeros(self.workspace_size(N), dtype=torch.uint8)


@pytest.fixture
def gpu_state(monkeypatch):
    state = types.SimpleNamespace(stream=0, capturing=False)
    monkeypatch.setattr(usp, "SparseMatrix", _Matrix)
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: state.capturing)
    monkeypatch.setattr(usp, "current_stream_handle", lambda: state.stream)
    return state


def _module():
    return linear.SparseLinear(torch.ones(4, 8), np.ones((4, 8), np.uint8), device=0)


@pytest.mark.parametrize("warm_up_stream", [0, 7])
def test_captured_buffer_is_kept_and_not_shared(gpu_state, warm_up_stream):
    mod = _module()
    gpu_state.stream = warm_up_stream
    mod.workspace(16)
    gpu_state.stream, gpu_state.capturing = 5, True
    captured = mod.workspace(16)
    assert mod.workspace(9) is captured  # a second call of the graph
    kept, ptr = weakref.ref(captured), captured.data_ptr()
    del captured
    gpu_state.stream, gpu_state.capturing = warm_up_stream, False
    eager = [mod.workspace(n) for n in (16, 1024, 16)]
    gc.collect()
    assert kept() is not None and kept().data_ptr() == ptr
    assert all(w is not kept() for w in eager)
    assert eager[1] is eager[2] and eager[1].numel() >= 100 * 1024


def test_buffer_of_a_capture_without_warm_up_is_not_used_eagerly(gpu_state):
    mod = _module()
    mod.workspace(16)
    gpu_state.capturing = True
    in_graph = mod.workspace(64)  # larger than anything a call left: cleared by the graph's replays only
    gpu_state.capturing = False
    assert mod.workspace(64) is not in_graph


def test_capture_while_another_thread_calls(gpu_state):
    mod = _module()
    mod.workspace(2)
    other = torch.zeros(100)

    class Small:  # looking at this buffer lets the other thread's first call on its stream run
        def numel(self):
            mod._ws[9] = other
            return 0

    mod._ws = {4: Small(), **mod._ws, 5: torch.zeros(1600)}
    warm = mod._ws[5]
    gpu_state.stream, gpu_state.capturing = 5, True
    assert mod.workspace(16) is warm
    assert 5 not in mod._ws and mod._ws[9] is other


def test_streams_do_not_share(gpu_state):
    mod = _module()
    first = mod.workspace(16)
    gpu_state.stream = 3
    second = mod.workspace(8)
    assert second is not first
    gpu_state.stream = 0
    assert mod.workspace(12) is first and mod.workspace(1) is None


@pytest.mark.gpu
def test_replay_after_the_workspace_has_grown():
    assert torch.cuda.is_available()
    g = torch.Generator(device="cuda").manual_seed(1)
    W = torch.randn(5120, 5120, generator=g, device="cuda", dtype=torch.float16)
    mod = linear.SparseLinear(W, torch.rand(5120, 5120, generator=g, device="cuda") < 0.5)
    x = torch.randn(16, 5120, generator=g, device="cuda", dtype=torch.float16)
    big = torch.randn(1024, 5120, generator=g, device="cuda", dtype=torch.float16)
    want = mod(x)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        y = mod(x)
    for i in range(4):
        want_big = mod(big[:1024 - 300 * i])  # a larger workspace the first time
        fill = [torch.full((1 << 20,), 0xAB, dtype=torch.uint8, device="cuda") for _ in range(64)]
        y.fill_(float("nan"))
        graph.replay()
        again = mod(big[:1024 - 300 * i])
        torch.cuda.synchronize()
        assert torch.equal(y.view(torch.int16), want.view(torch.int16))
        assert torch.equal(again.view(torch.int16), want_big.view(torch.int16))
        assert all(bool((f == 0xAB).all()) for f in fill)  # nothing was written into other tensors' memory
        del fill
