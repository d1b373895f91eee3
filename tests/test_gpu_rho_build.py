"""rho from the positions (ewald_energy_batch, and the FP32-mixed form's
rebuilds by the per-step calls and the fused sweep) against the direct sum
sum_p q_p exp(2 pi i n.s_p) in numpy, entry by entry in the storage order.

Sizes around the edges of the matrix-product build: 1 to 17 groups of 16
column pieces (one to all waves per group, one pass or several), columns cut
into pieces (longer than 24 entries), particle counts around multiples of four
and of the largest tile.

Tolerance, from the arithmetic and before any run: a phase is a product of at
most three table entries, each 8 multiplications (at 2 ulp) from a start whose
argument n s carries half an ulp of n turns; so an entry is off by at most
3 (16 + 2 pi n) + 4 roundings, and the sum by as many times sum |q|, the
roundings of N additions in whatever order included (another N).
"""
import math

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2507_02888_amd import ewald as ew
from paper_2507_02888_amd import workloads as wl

pytestmark = pytest.mark.gpu

# dim, particles, cutoff in units of 2 pi / L
SHAPES = [(3, 1, 2.1), (3, 2, 3.3), (3, 5, 5.2), (3, 63, 6.9), (3, 65, 8.0), (3, 130, 12.4),
          (2, 1, 1.2), (2, 3, 6.0), (2, 64, 15.0), (2, 67, 34.0)]


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ew.load()


def system(dim, n, gmul):
    rng = np.random.default_rng([31, dim, n])
    lat = np.eye(3)
    lat[:dim, :dim] += rng.uniform(-0.15, 0.15, (dim, dim))
    lat[:dim, :dim] *= 7.0
    L = abs(np.linalg.det(lat[:dim, :dim])) ** (1.0 / dim)
    q = rng.choice([-1.0, 0.5, 2.0], n)
    ions = rng.uniform(0, 7, (2, dim)) if n % 2 else np.zeros((0, dim))
    return wl.System(f"rho{dim}_{n}", dim, lat, n, q, ions, np.array([1.5, -0.5])[:len(ions)], 5.0 / L, 0.3 * L,
                     gmul * 2 * math.pi / L)


def direct(h, s, frac):
    n = h.tables()["n"][:, :s.dim]
    r = np.exp(2j * np.pi * (n @ frac.T)) @ s.mobile_q
    if s.n_fixed:
        f = s.fixed_pos @ np.linalg.inv(s.lattice[:s.dim, :s.dim])
        r += np.exp(2j * np.pi * (n @ f.T)) @ s.fixed_q
    nm = np.abs(n).max()
    count = s.n_mobile + s.n_fixed
    tol = (3 * (16 + 2 * math.pi * nm) + 4 + count) * 2.0 ** -53 * (np.abs(s.mobile_q).sum() + np.abs(s.fixed_q).sum())
    return r, 4 * tol  # numpy's own phases are off by as much


@pytest.mark.parametrize("dim,n,gmul", SHAPES)
def test_rho_entries(dim, n, gmul):
    s = system(dim, n, gmul)
    W, S = 3, 4
    rng = np.random.default_rng([32, dim, n])
    pos = rng.uniform(-7, 14, (W, n, dim))
    k = rng.integers(0, n, (S, W)).astype(np.int32)
    new = rng.uniform(-7, 14, (S, W, dim))
    acc = np.ones((S, W), dtype=np.uint8)
    dev = "cuda"
    kt, nt, at = (torch.tensor(x, device=dev) for x in (k, new, acc))
    for prec in (ew.EWALD_FP64, ew.EWALD_FP32_MIXED):
        h = ew.System(s, precision=prec, refresh_every=2 if prec else 0)
        shapes = [None, {}] + ([{"threads": t} for t in (512, 1024) if h.info["n_slots"] // 4 <= 1024] if prec else [])
        for tune in shapes:  # None: the per-step calls
            b = ew.Batch([h], np.zeros(W, dtype=np.int32))
            e = torch.zeros(W, dtype=torch.float64, device=dev)
            d = torch.zeros((S, W), dtype=torch.float64, device=dev)
            b.energy(torch.tensor(pos.reshape(-1, dim), device=dev), e)
            torch.cuda.synchronize()
            for w in range(W):
                ref, tol = direct(h, s, b.walker_positions(w))
                assert np.max(np.abs(b.walker_rho(w) - ref)) <= tol
            if prec != ew.EWALD_FP32_MIXED:
                continue
            if tune is None:
                for m in range(S):
                    b.move_delta(kt[m], nt[m], d[m])
                    b.accept(at[m])
            else:
                try:
                    b.set_tuning(**tune)
                except ew.EwaldError:
                    continue  # not a workgroup size for this segment count
                b.run_moves(kt, nt, at, d)
            torch.cuda.synchronize()
            for w in range(W):  # rebuilt after the last move (S is a multiple of the refresh interval)
                ref, tol = direct(h, s, b.walker_positions(w))
                assert b.walker_header(w)["n_refresh"] == S // 2
                assert np.max(np.abs(b.walker_rho(w) - ref)) <= tol
