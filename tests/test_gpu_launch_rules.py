"""The fused sweep's shape for walkers of 512 to 1024 segments and particles, with nothing
fixed, where more walkers than compute units would fit two workgroups of 512
threads on each: taken by one-plane systems, and not where those kernels spill (two
planes; the u term in two dimensions in FP64), which keep 1024 threads."""
import math

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2507_02888_amd import ewald as ew
from paper_2507_02888_amd import workloads as wl

pytestmark = pytest.mark.gpu
FP64, MIXED = ew.EWALD_FP64, ew.EWALD_FP32_MIXED


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ew.load()


def system(kind):
    if kind.startswith("bilayer"):
        s = wl.bilayer(300)
        s.g_cut = 38 * 2 * math.pi / s.length
        return s
    s = wl.config(3).systems[0] if kind.startswith("hex") else wl.config(5).systems[0]
    if kind.startswith("hex"):
        n = 600
        L = math.sqrt(math.pi * 25 * n)
        s = wl.System("hex600", 2, wl.hex_cell(math.pi * 25 * n), n, -np.ones(n), np.zeros((0, 2)), np.zeros(0), 5 / L,
                      0.5 * L, 40 * 2 * math.pi / L)
    return wl.with_u_term(s, 3 if s.dim == 2 else 5) if kind.endswith("_u") else s


@pytest.mark.parametrize("precision", [FP64, MIXED], ids=["fp64", "mixed"])
@pytest.mark.parametrize("kind,threads", [("bcc", (512, 512)), ("bcc_u", (512, 512)), ("hex", (512, 512)),
                                          ("hex_u", (1024, 512)), ("bilayer", (1024, 1024))])
def test_large_walker_shape(kind, threads, precision):
    s = system(kind)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    h = ew.System(s, precision=precision, refresh_every=4 if precision == MIXED else 0)
    assert 512 < h.info["n_slots"] // 4 <= 1024 and 512 < s.n_mobile <= 1024
    few, many = ew.Batch([h], np.zeros(cus, np.int32)), ew.Batch([h], np.zeros(cus + 1, np.int32))
    assert few.tuning()["threads"] == 1024
    t = many.tuning()
    assert t["fused"] == 1 and t["threads"] == threads[0 if precision == FP64 else 1]
    assert t["waves"] == (4 if t["threads"] == 512 else 0)
