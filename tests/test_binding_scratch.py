"""Scratch memory that the binding allocates by itself belongs to one call and to the stream that the call's kernels run
on (no GPU: the library, the stream context and the allocator are replaced by recorders)."""
import contextlib
import types

import pytest
import torch

from paper_2512_07011_amd import binding


class Recorder:
    """Stands for the library: every entry point succeeds; forward calls leave (workspace address, stream)."""

    def __init__(self):
        self.calls = []

    def bsfa_forward_workspace_bytes(self, pref):
        return 4096

    bsfa_calibrate_workspace_bytes = bsfa_forward_workspace_bytes

    def bsfa_forward(self, pref, q, k, v, tau, causal, out, st, stream):
        self.calls.append((pref._obj.workspace, stream))
        return 0

    def bsfa_calibrate(self, pref, q, k, causal, fr, n, out, ws, nbytes, stream):
        self.calls.append((ws, stream.value))
        return 0

    def bsfa_calibrate_topk(self, pref, q, k, causal, ks, n, done, out, ws, nbytes, stream):
        self.calls.append((ws, stream.value))
        return 0


@pytest.fixture
def recorded(monkeypatch):
    lib, made, inside = Recorder(), [], [1]                    # 1: the current stream
    empty = torch.empty

    def record_empty(*a, **kw):
        t = empty(*a, **kw)
        made.append((t, inside[-1]))                           # (kept alive: no address is handed out twice)
        return t

    @contextlib.contextmanager
    def stream_context(s):
        inside.append(s.cuda_stream)
        yield
        inside.pop()

    monkeypatch.setattr(binding, "lib", lambda: lib)
    monkeypatch.setattr(binding, "_dev_check", lambda *ts: None)
    monkeypatch.setattr(binding, "_raw_stream", lambda s, device: 1 if s is None else s.cuda_stream)
    monkeypatch.setattr(torch, "empty", record_empty)
    monkeypatch.setattr(torch.cuda, "stream", stream_context)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device=None: types.SimpleNamespace(cuda_stream=1))
    return lib, made


def test_scratch_belongs_to_the_call_and_to_its_stream(recorded):
    lib, made = recorded
    q = torch.zeros(1, 128, 2, 128, dtype=torch.bfloat16)
    streams = [None, types.SimpleNamespace(cuda_stream=2), types.SimpleNamespace(cuda_stream=3), None]
    for s in streams:
        binding.bsfa_forward(q, q, q, torch.zeros(2), out=q, stream=s)
        binding.bsfa_calibrate(q, q, [0.5], stream=s)
        binding.bsfa_calibrate_topk([(q, q)], [1], stream=s)
    assert len(lib.calls) == 12 and len({ws for ws, _ in lib.calls}) == 12          # no two calls share scratch memory
    allocated_on = {t.data_ptr(): s for t, s in made}
    for ws, launched_on in lib.calls:
        assert allocated_on[ws] == launched_on


def test_stream_without_the_quick_query(monkeypatch):
    """Where torch lacks its unofficial query for the current stream, the public one answers."""
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device=None: types.SimpleNamespace(cuda_stream=77))
    assert binding._raw_stream(None, torch.device("cuda", 0)) == 77
    assert binding._raw_stream(types.SimpleNamespace(cuda_stream=5), torch.device("cuda", 0)) == 5


@pytest.mark.parametrize("shape", [(128, 128), (1, 128, 2)])
def test_forward_refuses_tensors_that_are_not_four_dimensional(recorded, shape):
    q = torch.zeros(shape, dtype=torch.bfloat16)
    for tau in (torch.zeros(2), torch.zeros(128)):
        with pytest.raises(ValueError):
            binding.bsfa_forward(q, q, q, tau, out=q)
