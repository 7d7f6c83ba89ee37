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


class Density:
    """The library's sizes, and a deposit that only looks at its workspace."""

    def __init__(self):
        self.library, self.held = ndgp.lib(), None

    def __getattr__(self, name):
        return getattr(self.library, name)

    def ndgp_cic_density(self, grid, pos, count, delta, ws, ws_bytes, stream):
        self.held = ws_bytes
        return ndgp.NDGP_OK


@pytest.mark.parametrize("n,m,count,extra", [
    (256, 0, 1000, 0), (32, 32, 1000, 0), (256, 128, 311295, 0),  # no level sorted
    (32, 0, 60000, 24 * 60000 + (1 << 19)),  # sorted: the particles, a table of 64 tiles
    (64, 32, 1 << 26, (24 << 20) + (1 << 22)),  # a chunk of them at a time
])
def test_cic_density_holds_the_scratch_it_can_use(on_host, n, m, count, extra):
    """The workspace of a deposit: the accumulators, and scratch for as many particles
    as are sorted (guard bands and alignment of seven buffers aside)."""
    lib = Density()
    on_host.setattr(ndgp, "lib", lambda: lib)
    grid = ndgp.Grid(n=n, h=1.0, patches=[ndgp.Patch(m, (2, 2, 2))] if m else [])
    pos = torch.empty((3, count), dtype=torch.float64, device="meta")
    on_host.setattr(ndgp, "_dev", lambda t, shape=None, name="": 0)
    delta = [torch.empty(1, dtype=torch.float64)] * (2 if m else 1)
    on_host.setattr(ndgp, "workspace", lambda nbytes, device, stream: torch.empty(nbytes, dtype=torch.uint8))
    ndgp.cic_density(grid, pos, delta=delta)
    least = 8 * (n**3 + m**3)
    assert least <= lib.held <= least + extra + 7 * 1024
    assert lib.held <= lib.library.ndgp_cic_workspace_bytes(grid._c())
