"""rho of walkers of few particles (built by segments) and of more (by groups of column
pieces), in one plane and two, with and without ions, against the direct sum
sum_p q_p exp(2 pi i n.s_p) in numpy, entry by entry: by the energy call, and by the
per-step rebuild of batches whose workgroups take several walkers each, some of them
due and some not.  Sizes on both sides of the rule (40, and 64 with 97 to 256
segments) and of whole fours of particles.

Tolerance, from the arithmetic and before any run: a phase is a product of at
most three table entries, each 8 multiplications (2 ulp) from a start whose argument
n s carries half an ulp of n turns, so an entry is off by at most 3 (16 + 2 pi n) + 4
roundings, and the sum by as many times sum |q|, with N more for the additions;
four times that, as numpy's own phases are off by as much.
"""
import math

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2507_02888_amd import ewald as ew
from paper_2507_02888_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ew.load()


def system(dim, n, gmul, planes=1, ions=0):
    rng = np.random.default_rng([61, dim, n])
    lat = np.eye(3)
    lat[:dim, :dim] = 7.0 * (np.eye(dim) + rng.uniform(-0.15, 0.15, (dim, dim)))
    L = abs(np.linalg.det(lat[:dim, :dim])) ** (1.0 / dim)
    s = wl.System(f"seg{dim}_{n}", dim, lat, n, rng.choice([-1.0, 0.5, 2.0], n), rng.uniform(0, 7, (ions, dim)),
                  rng.choice([1.5, -0.5], ions), 5.0 / L, 0.3 * L, gmul * 2 * math.pi / L)
    if planes == 2:
        n0 = (n + 1) // 3
        s.layer_z = np.array([0.0, 1.5])
        s.mobile_layer = (np.arange(n) >= n0).astype(np.int32)
        s.fixed_layer = (np.arange(ions) % 2).astype(np.int32)
    return s


def direct(h, s, frac, plane):
    """rho of one plane and its tolerance."""
    n = h.tables()["n"][:, :s.dim]
    own = np.ones(s.n_mobile, bool) if s.layer_z is None else s.mobile_layer == plane
    ion = np.ones(s.n_fixed, bool) if s.layer_z is None else s.fixed_layer == plane
    r = np.exp(2j * np.pi * (n @ frac[own].T)) @ s.mobile_q[own]
    if ion.any():
        f = s.fixed_pos[ion] @ np.linalg.inv(s.lattice[:s.dim, :s.dim])
        r = r + np.exp(2j * np.pi * (n @ f.T)) @ s.fixed_q[ion]
    q = np.abs(s.mobile_q).sum() + np.abs(s.fixed_q).sum()
    return r, 4 * (3 * (16 + 2 * math.pi * np.abs(n).max()) + 4 + s.n_mobile + s.n_fixed) * 2.0 ** -53 * q


CASES = [(3, 1, 5.0, 1, 0), (3, 2, 11.0, 1, 2), (3, 7, 8.0, 1, 0), (3, 40, 7.0, 1, 3), (3, 41, 8.0, 1, 0), (3, 54, 6.0, 1, 0),
         (3, 64, 7.0, 1, 1), (3, 65, 7.0, 1, 0), (2, 1, 3.0, 1, 1), (2, 8, 34.0, 1, 0), (2, 39, 16.0, 1, 2),
         (2, 64, 16.0, 1, 0), (2, 3, 10.0, 2, 0), (2, 40, 16.0, 2, 3), (2, 41, 6.0, 2, 0), (2, 64, 16.0, 2, 2),
         (2, 90, 16.0, 2, 0)]


@pytest.mark.parametrize("dim,n,gmul,planes,ions", CASES)
def test_energy_rho(oracle_lib, dim, n, gmul, planes, ions):
    s = system(dim, n, gmul, planes, ions)
    h = ew.System(s)
    W = 3
    b = ew.Batch([h], np.zeros(W, np.int32))
    rng = np.random.default_rng([62, dim, n])
    pos = rng.uniform(-7, 14, (W, n, dim))
    e = torch.zeros(W, dtype=torch.float64, device="cuda")
    b.energy(torch.tensor(pos.reshape(-1, dim), device="cuda"), e)
    torch.cuda.synchronize()
    for w in range(W):
        for p in range(planes):
            ref, tol = direct(h, s, b.walker_positions(w), p)
            assert np.max(np.abs(b.walker_rho(w, p) - ref)) <= tol, (w, p)
        ref = oracle_lib.energy(s, *oracle_lib.particles(s, pos[w]))["total"]
        scale = max(abs(ref), s.alpha / math.sqrt(math.pi) * float((s.mobile_q ** 2).sum() + (s.fixed_q ** 2).sum()))
        assert abs(float(e[w]) - ref) <= 1e-10 * scale


@pytest.mark.parametrize("n,gmul,planes", [(12, 5.0, 1), (64, 7.0, 1), (70, 5.0, 1), (30, 16.0, 2), (90, 12.0, 2)])
@pytest.mark.parametrize("W", [1030, 9000])
def test_step_rebuilds_of_many_walkers(W, n, gmul, planes):
    dim = 3 if planes == 1 else 2
    s = system(dim, n, gmul, planes, 0)
    S, K = 7, 2
    rng = np.random.default_rng([63, W, n])
    h = ew.System(s, precision=ew.EWALD_FP32_MIXED, refresh_every=K)
    b = ew.Batch([h], np.zeros(W, np.int32))
    f = dict(device="cuda")
    acc = (rng.random((S, W)) < rng.choice([0.0, 0.3, 0.9], W)).astype(np.uint8)
    k, new = rng.integers(0, n, (S, W)).astype(np.int32), rng.uniform(-7, 14, (S, W, dim))
    pos = torch.tensor(rng.uniform(-7, 14, (W * n, dim)), **f)
    kt, nt, at = (torch.tensor(x, **f) for x in (k, new, acc))
    e, d = torch.zeros(W, dtype=torch.float64, **f), torch.zeros((S, W), dtype=torch.float64, **f)
    b.energy(pos, e)
    for m in range(S):
        b.move_delta(kt[m], nt[m], d[m])
        b.accept(at[m])
    torch.cuda.synchronize()
    size = b.state_bytes // W
    ints = b.state.view(W, size)[:, :16].cpu().numpy().view(np.int32)  # counter, pending, accepts, rebuilds
    accepts = acc.sum(0)
    assert np.array_equal(ints[:, 2], accepts)
    assert np.array_equal(ints[:, 3], accepts // K)
    fresh = np.nonzero((accepts > 0) & (accepts % K == 0))[0]  # rho as last rebuilt (no accept since)
    assert len(fresh) > 100 and (accepts == 0).sum() > 100 and (accepts % K == 1).sum() > 100
    for w in list(fresh[:20]) + list(fresh[-20:]) + list(np.nonzero(accepts == 0)[0][:10]):
        for p in range(planes):
            ref, tol = direct(h, s, b.walker_positions(int(w)), p)
            assert np.max(np.abs(b.walker_rho(int(w), p) - ref)) <= tol, (w, p)


@pytest.mark.parametrize("sizes", [((12, 5.0), (40, 9.0)), ((12, 5.0), (90, 9.0)), ((3, 11.0), (64, 7.0), (33, 4.0)),
                                   ((3, 11.0), (65, 7.0), (300, 4.0))])
def test_systems_in_one_batch(oracle_lib, sizes):
    """Systems of several sizes and cutoffs together: all of few particles, and beside larger ones."""
    K, S, reps = 2, 4, 3
    ss = [system(3, n, g, 1, i) for i, (n, g) in enumerate(sizes)]
    hs = [ew.System(s, precision=ew.EWALD_FP32_MIXED, refresh_every=K) for s in ss]
    which = np.tile(np.arange(len(ss), dtype=np.int32), reps)
    W, f = len(which), dict(device="cuda")
    b = ew.Batch(hs, which)
    rng = np.random.default_rng([64, len(ss), ss[1].n_mobile])
    pos = [rng.uniform(-7, 14, (ss[i].n_mobile, 3)) for i in which]
    e, d = torch.zeros(W, dtype=torch.float64, **f), torch.zeros(W, dtype=torch.float64, **f)
    b.energy(torch.tensor(np.concatenate(pos), **f), e)
    torch.cuda.synchronize()
    for w, i in enumerate(which):
        ref, tol = direct(hs[i], ss[i], b.walker_positions(w), 0)
        assert np.max(np.abs(b.walker_rho(w) - ref)) <= tol, w
        ref = oracle_lib.energy(ss[i], *oracle_lib.particles(ss[i], pos[w]))["total"]
        scale = max(abs(ref), ss[i].alpha / math.sqrt(math.pi) * float((ss[i].mobile_q ** 2).sum() + (ss[i].fixed_q ** 2).sum()))
        assert abs(float(e[w]) - ref) <= 1e-10 * scale
    for m in range(S):  # every walker due after the second and the fourth
        k = np.array([rng.integers(ss[i].n_mobile) for i in which], np.int32)
        b.move_delta(torch.tensor(k, **f), torch.tensor(rng.uniform(-7, 14, (W, 3)), **f), d)
        b.accept(torch.ones(W, dtype=torch.uint8, **f))
    torch.cuda.synchronize()
    for w, i in enumerate(which):
        ref, tol = direct(hs[i], ss[i], b.walker_positions(w), 0)
        assert np.max(np.abs(b.walker_rho(w) - ref)) <= tol, w
