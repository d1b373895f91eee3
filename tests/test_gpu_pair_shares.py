"""ewald_energy_batch against the oracle at particle counts around the edges of
the pair loop: no whole group of four partners, one to eight shares of a
particle's partners (from 1 to more items than threads), odd and even counts, with
and without fixed ions and the u term; two walkers.

Tolerance, from before any run: 1e-10 of the energy or of the self energy sum q^2 alpha / sqrt(pi)
(the charges of both signs cancel in the energy), the bound that the energies of the
workloads are held to (the polynomial's fit is 1e-12, and below 10^5 roundings
of 1.1e-16 of terms that are no larger add 1e-11).
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


def system(dim, n, ions, skew, alpha_l):
    rng = np.random.default_rng([23, dim, n])
    L = (4.0 * n) ** (1.0 / dim) + 2.0
    lat = np.eye(3)
    lat[:dim, :dim] *= L
    if skew:
        lat[:dim, :dim] += np.triu(rng.uniform(-0.1, 0.1, (dim, dim)) * L, 1)
    q = rng.choice([-1.0, 0.5], n)
    f = rng.uniform(0, L, (ions, dim))
    return wl.System(f"pairs{dim}_{n}", dim, lat, n, q, f, rng.choice([1.0, -2.0], ions), alpha_l / L, 0.4 * L,
                     12.0 / L)


@pytest.mark.parametrize("u", [False, True], ids=["p", "pu"])
@pytest.mark.parametrize("dim,skew,alpha_l", [(3, False, 5.0), (3, True, 5.0), (2, False, 5.0), (3, False, 9.0)])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 7, 8, 9, 10, 32, 33, 54, 85, 86, 127, 128, 129, 200, 255, 256, 257, 300, 512])
def test_energy_at_share_edges(oracle_lib, n, dim, skew, alpha_l, u):
    s = system(dim, n, 3 if n % 3 == 0 else 0, skew, alpha_l)
    if u:
        s = wl.with_u_term(s, 1)
    print(f"[pairs] n={n} dim={dim} skew={skew} alpha L={alpha_l} u={u}", flush=True)
    ja = np.random.default_rng(3).uniform(-0.01, 0.01, 2048)
    h = ew.System(s, jastrow_a=ja)
    b = ew.Batch([h], np.zeros(2, np.int32))
    pos = np.random.default_rng([5, n]).random((2, n, dim)) @ s.lattice[:dim, :dim]
    e, j = (torch.zeros(2, dtype=torch.float64, device="cuda") for _ in range(2))
    b.energy(torch.tensor(pos.reshape(-1, dim), device="cuda"), e, j)
    torch.cuda.synchronize()
    for w in range(2):
        ref = oracle_lib.energy(s, *oracle_lib.particles(s, pos[w]), jastrow_a=ja)
        scale = max(1.0, abs(ref["total"]), float((s.mobile_q ** 2).sum()) * s.alpha / math.sqrt(math.pi))
        assert math.isfinite(float(e[w]))
        assert abs(float(e[w]) - ref["total"]) <= 1e-10 * scale, w
        assert abs(float(j[w]) - ref["jastrow"]) <= 1e-10 * max(1.0, abs(ref["jastrow"])), w
