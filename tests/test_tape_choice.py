"""Whether an optimisation step keeps an adjoint tape: every step of a loop
decides like the first, whatever torch's allocator and the library keep idle
from the steps before.  The device is a stand-in: 288 GB, its idle memory told
by the three calls that the decision asks."""
import contextlib

import pytest
import torch

from paper_1410_1629_amd import autograd, binding

GB = 10 ** 9


class _Device:
    """free: of the device; cached: idle in torch's allocator; kept: idle in the library."""

    def __init__(self, monkeypatch, free, cached, kept, need):
        self.free, self.cached, self.kept, self.released = free, cached, kept, 0
        monkeypatch.setattr(torch.cuda, "device", lambda d: contextlib.nullcontext())
        monkeypatch.setattr(torch.cuda, "mem_get_info", lambda *a: (self.free, 288 * GB))
        monkeypatch.setattr(torch.cuda, "memory_reserved", lambda *a: self.cached + 5 * GB)
        monkeypatch.setattr(torch.cuda, "memory_allocated", lambda *a: 5 * GB)
        monkeypatch.setattr(binding, "kept_bytes", lambda: self.kept, raising=False)
        monkeypatch.setattr(binding, "release_workspaces", self._release)
        monkeypatch.setattr(binding, "tape_bytes", lambda prob, **kw: need)
        monkeypatch.setattr(torch, "empty", self._empty)

    def _release(self):
        self.free, self.kept, self.released = self.free + self.kept, 0, self.released + 1

    def _empty(self, n, dtype, device):
        if n > self.free + self.cached:
            raise torch.cuda.OutOfMemoryError("out of memory")
        return "tape of %d" % n


@pytest.mark.parametrize("need", [10 * GB, 50 * GB, 60 * GB, 69 * GB])
def test_a_later_step_decides_like_the_first(monkeypatch, need):
    first = _Device(monkeypatch, 280 * GB, 0, 0, need)
    assert autograd._tape_for({}, "cuda:0") == "tape of %d" % need
    # the first step's tape is in torch's cache, its workspaces are kept
    later = _Device(monkeypatch, 280 * GB - need - 64 * GB, need, 64 * GB, need)
    assert autograd._tape_for({}, "cuda:0") == "tape of %d" % need
    assert first.released == later.released == 0


def test_too_large_a_tape_is_never_made(monkeypatch):
    _Device(monkeypatch, 280 * GB, 0, 0, 71 * GB)
    assert autograd._tape_for({}, "cuda:0") is None
    _Device(monkeypatch, 100 * GB, 116 * GB, 64 * GB, 71 * GB)
    assert autograd._tape_for({}, "cuda:0") is None


def test_kept_memory_makes_room(monkeypatch):
    dev = _Device(monkeypatch, 10 * GB, 0, 64 * GB, 17 * GB)
    assert autograd._tape_for({}, "cuda:0") == "tape of %d" % (17 * GB)
    assert dev.released == 1 and dev.kept == 0


def test_no_tape_where_torchs_memory_is_in_pieces(monkeypatch):
    dev = _Device(monkeypatch, 200 * GB, 0, 0, 40 * GB)

    def pieces(*a, **kw):
        raise torch.cuda.OutOfMemoryError("out of memory")

    monkeypatch.setattr(torch, "empty", pieces)
    assert autograd._tape_for({}, "cuda:0") is None and dev.released == 0
