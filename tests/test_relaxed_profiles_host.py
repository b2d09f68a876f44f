"""Fitting the profiles of many lattices keeps a bounded amount of density fields alive: 64 MiB
of them, or one that is larger by itself (CPU, with a stand-in for the batch)."""
import gc
import weakref

import pytest

torch = pytest.importorskip("torch")
from paper_1211_6932_amd import initialiser as I  # noqa: E402
from paper_1211_6932_amd import lbmp  # noqa: E402


class Field:
    def record_stream(self, stream):
        pass


class Stream:
    cuda_stream = 0

    def synchronize(self):
        pass


class FakeBatch:
    device, stream = torch.device("cpu"), Stream()

    def __init__(self):
        self.alive, self.most = [], 0

    def moments(self, i):
        f = Field()
        self.alive = [r for r in self.alive if r() is not None] + [weakref.ref(f)]
        self.most = max(self.most, len(self.alive))
        return f, None, None


class Lattice:
    def __init__(self, n):
        self.params, self.info = dict(nx=n, ny=n), dict(cx=0.5 * n, cy=0.5 * n, R0=0.2 * n)


@pytest.mark.parametrize("side,n,at_once", [(8192, 5, 1), (4096, 6, 1), (2048, 12, 4), (256, 96, 32)])
def test_density_fields_alive(side, n, at_once, monkeypatch):
    calls = []

    def extract(rhos, places, out, scratch, stream=0):
        calls.append(len(rhos))
        out.fill_(len(calls))
        return out

    monkeypatch.setattr(lbmp, "profiles_extract", extract)
    gc.collect()
    batch = FakeBatch()
    out = I.relaxed_profiles(batch, [Lattice(side)] * n, range(n))
    assert sum(calls) == n and max(calls) == min(at_once, n)
    assert batch.most <= 2 * at_once  # those of this call, and of the last one until they are replaced
    assert out.shape == (n, 128) and float(out[-1, 0]) == len(calls)
