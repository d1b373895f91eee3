"""The fused sweep at 512 and 1024 threads where walkers have more than 512
segments of the structure factor, for walkers below and above 512 particles, in
one plane and in two: the kernel runs (no fall-back to the per-step calls), its
deltas agree with theirs, and in the mixed form rho after a rebuild agrees entry
by entry with the direct sum sum_p q_p exp(2 pi i n.s_p) in numpy.

Tolerances, from before any run.  FP64 deltas: sums in another order, 1e-12 of
the energy or of the largest delta (10^4 roundings of 1.1e-16).  Mixed deltas: each path is
held to 1e-5 Ha of the exact value, so they are within 2e-5 of each other.  rho:
a phase is a product of at most three table entries, each 8 multiplications (2 ulp)
from a start whose argument n s carries half an ulp of n turns, so an entry is off by
at most 3 (16 + 2 pi n) + 4 roundings and the sum by as many times sum |q|, N
more for the additions; four times that, as numpy's own phases are off by as much.
"""
import math

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2507_02888_amd import ewald as ew
from paper_2507_02888_amd import workloads as wl

pytestmark = pytest.mark.gpu

# cell, particles, cutoff in units of 2 pi / L, segments from and up to, shapes
CASES = [("sc", 60, 10.5, 512, 1024, (0, 512, 1024)), ("bcc", 600, 10.5, 512, 1024, (0, 512, 1024)),
         ("sc", 512, 12.7, 1024, 2048, (0, 512)), ("sc", 130, 12.7, 1024, 2048, (0, 512)),
         ("fcc", 513, 12.7, 1024, 2048, (0, 512)), ("hex", 100, 44.0, 512, 1024, (0, 512, 1024)),
         ("bilayer", 90, 44.0, 512, 1024, (0, 512, 1024)), ("bilayer", 600, 44.0, 512, 1024, (0, 512, 1024)),
         ("bilayer", 40, 60.0, 1024, 2048, (0, 512))]


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ew.load()


def system(cell, n, gmul):
    if cell == "bilayer":
        s = wl.bilayer(n // 2, 2.0, 1.0)
        L = s.length
        s.g_cut = gmul * 2 * math.pi / L
        return s
    dim = 2 if cell == "hex" else 3
    lat = {"sc": wl.sc_cell, "fcc": wl.fcc_cell, "bcc": wl.bcc_cell, "hex": wl.hex_cell}[cell](4.0 * n)
    L = (4.0 * n) ** (1.0 / dim)
    rc = min(0.5 * L, 0.999 * wl.inscribed_radius(cell, 4.0 * n))
    return wl.System(f"{cell}{n}", dim, lat, n, -np.ones(n), np.zeros((0, dim)), np.zeros(0), 5.0 / L, rc,
                     gmul * 2 * math.pi / L)


@pytest.mark.parametrize("cell,n,gmul,above,upto,shapes", CASES)
@pytest.mark.parametrize("precision", [ew.EWALD_FP64, ew.EWALD_FP32_MIXED], ids=["fp64", "mixed"])
def test_fused_large_segment_counts(cell, n, gmul, above, upto, shapes, precision):
    s = system(cell, n, gmul)
    d, W, S = s.dim, 2, 10
    mixed = precision == ew.EWALD_FP32_MIXED
    rng = np.random.default_rng([47, n])
    lat = s.lattice[:d, :d]
    k = rng.integers(0, n, (S, W)).astype(np.int32)
    f = dict(device="cuda")
    pos = torch.tensor((rng.random((W, n, d)) @ lat).reshape(-1, d), **f)
    kt, nt, at = torch.tensor(k, **f), torch.tensor(rng.random((S, W, d)) @ lat, **f), torch.ones((S, W), dtype=torch.uint8, **f)
    h = ew.System(s, precision=precision, refresh_every=5 if mixed else 0)
    assert above < h.info["n_slots"] // 4 <= upto

    def run(threads):
        b = ew.Batch([h], np.zeros(W, dtype=np.int32))
        e = torch.zeros(W, dtype=torch.float64, **f)
        out = torch.zeros((S, W), dtype=torch.float64, **f)
        b.energy(pos, e)
        if threads is None:
            for m in range(S):
                b.move_delta(kt[m], nt[m], out[m])
                b.accept(at[m])
        else:
            b.set_tuning(threads=threads)
            t = b.tuning()
            assert t["fused"] == 1 and t["threads"] in ((threads,) if threads else (512, 1024))
            b.run_moves(kt, nt, at, out)
        torch.cuda.synchronize()
        return b, e.cpu().numpy(), out.cpu().numpy()

    _, e0, ref = run(None)
    scale = max(1.0, float(np.abs(e0).max()), float(np.abs(ref).max()))
    idx = h.tables()["n"][:, :d]
    nm = float(np.abs(idx).max())
    q = np.abs(s.mobile_q).sum()
    tol_rho = 4 * (3 * (16 + 2 * math.pi * nm) + 4 + n) * 2.0 ** -53 * q
    for threads in shapes:
        b, _, got = run(threads)
        err = float(np.max(np.abs(got - ref)))
        print(f"[large] {cell}{n} threads={threads} deltas {err:.2e}", flush=True)
        assert err <= (2e-5 if mixed else 1e-12 * scale)
        for w in range(W):
            if mixed:
                assert b.walker_header(w)["n_refresh"] == S // 5
            frac = b.walker_positions(w)
            planes = [np.ones(n, bool)] if s.layer_z is None else [s.mobile_layer == 0, s.mobile_layer == 1]
            for p, own in enumerate(planes):
                direct = np.exp(2j * np.pi * (idx @ frac[own].T)) @ s.mobile_q[own]
                worst = float(np.max(np.abs(b.walker_rho(w, p) - direct)))
                # (in the FP64 form rho carries S updates instead of a rebuild: each within one entry's bound)
                assert worst <= tol_rho * (1 if mixed else S + 1), (threads, w, p, worst, tol_rho)
