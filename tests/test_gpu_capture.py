"""Batches and systems dropped while a stream is being captured: the capture
goes on, and its graph replays as the eager calls run."""
import gc
import threading

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2507_02888_amd import ewald as ew
from paper_2507_02888_amd import workloads as wl

pytestmark = pytest.mark.gpu
W, S = 3, 6


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ew.load()


class Walkers:
    def __init__(self, seed):
        s = wl.config(2).systems[0]
        rng = np.random.default_rng([43, seed])
        lat = s.lattice
        self.sys = ew.System(s, precision=ew.EWALD_FP32_MIXED, refresh_every=2)
        self.batch = ew.Batch([self.sys], np.zeros(W, np.int32))
        f = dict(device="cuda")
        self.pos = torch.tensor((rng.random((W, s.n_mobile, 3)) @ lat).reshape(-1, 3), **f)
        self.k = torch.tensor(rng.integers(0, s.n_mobile, (S, W)).astype(np.int32), **f)
        self.new = torch.tensor(rng.random((S, W, 3)) @ lat, **f)
        self.acc = torch.tensor(rng.integers(0, 2, (S, W)).astype(np.uint8), **f)
        self.e = torch.zeros(W, dtype=torch.float64, **f)
        self.d = torch.zeros((S, W), dtype=torch.float64, **f)

    def block(self):
        self.batch.energy(self.pos, self.e)
        self.batch.run_moves(self.k, self.new, self.acc, self.d)

    def drop(self):
        self.batch.close()
        self.sys.close()


def drop_at_once(w):
    w.drop()


def drop_by_collection(w):
    w.batch.cycle, w.sys.cycle = w.batch, w.sys  # reachable from themselves alone, once w lets go
    del w.batch, w.sys
    gc.collect()


def drop_on_another_thread(w):
    t = threading.Thread(target=w.drop)
    t.start()
    t.join()


@pytest.mark.parametrize("drop", [drop_at_once, drop_by_collection, drop_on_another_thread])
def test_dropped_during_a_capture(drop):
    kept, dropped = Walkers(1), Walkers(2)
    for w in (kept, dropped):
        w.block()
    torch.cuda.synchronize()
    ref = kept.e.clone(), kept.d.clone()
    gc.collect()  # what other tests left
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        kept.batch.energy(kept.pos, kept.e)
        drop(dropped)
        kept.batch.run_moves(kept.k, kept.new, kept.acc, kept.d)
    for _ in range(3):
        kept.e.zero_()
        kept.d.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(kept.e, ref[0]) and torch.equal(kept.d, ref[1])
        Walkers(3).block()  # eager work, in memory that may be the dropped ones'
        torch.cuda.synchronize()
