"""Scratch buffers of the Python calls, against a library that only records what it
is handed (no GPU)."""
import contextlib
import types

import pytest
import torch

from paper_1511_08200_amd import ndgp


class Recorder:
    """Stands for the library: answers the size questions, keeps the workspaces."""

    def __init__(self, nbytes, during=None):
        self.nbytes, self.during, self.calls = nbytes, during, []

    def ndgp_cic_force_workspace_bytes(self, grid, count):
        return self.nbytes

    def ndgp_cic_force_in(self, grid, force, pos, count, out, ws, ws_bytes, stream):
        self.calls.append((ws, ws_bytes))
        if self.during:  # another caller's turn while this call's workspace is in use
            self.during, again = None, self.during
            again()
        return ndgp.NDGP_OK


@pytest.fixture
def on_host(monkeypatch):
    monkeypatch.setattr(ndgp, "_dev", lambda t, shape=None, name="": t.data_ptr())
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(torch.cuda, "current_stream",
                        lambda device=None: types.SimpleNamespace(cuda_stream=0))
    monkeypatch.setattr(torch.cuda, "stream", lambda s: contextlib.nullcontext())
    monkeypatch.setattr(ndgp, "_ws_cache", {})
    return monkeypatch


def _call():
    grid = ndgp.Grid(n=8, h=1.0)
    force = [torch.zeros((3, 8, 8, 8), dtype=torch.float64)]
    return ndgp.cic_force(grid, force, torch.zeros((3, 5), dtype=torch.float64))


def test_cic_force_has_scratch_of_its_own(on_host):
    """Two calls on one stream at a time (two host threads) never hold one buffer,
    and nothing is kept once they have returned."""
    lib = Recorder(4096, during=_call)
    on_host.setattr(ndgp, "lib", lambda: lib)
    _call()
    (a, na), (b, nb) = lib.calls
    assert na >= 4096 and nb >= 4096 and a != b
    assert not ndgp._ws_cache


def test_cic_force_runs_without_room_for_scratch(on_host):
    lib = Recorder(1 << 20)
    on_host.setattr(ndgp, "lib", lambda: lib)
    empty = torch.empty

    def no_room(*args, dtype=None, **kw):
        if dtype == torch.uint8:
            raise torch.OutOfMemoryError("no room")
        return empty(*args, dtype=dtype, **kw)

    on_host.setattr(torch, "empty", no_room)
    _call()
    assert lib.calls == [(None, 0)]
