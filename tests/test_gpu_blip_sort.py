"""Blip batches in the range that is served in the order of the points' places on
the grid (16 MB of coefficients and half a gigabyte of rows at least), against
the same points in small calls, which are not: each point's arithmetic is the same,
so every output is bit for bit the same.  Points spread over the cell, all in one
brick of the grid, and half in one brick; and points in one brick take no longer
than three times as long as spread ones."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2507_02888_amd import ewald as ew

pytestmark = pytest.mark.gpu

LAT = np.array([[9.0, 0.2, 0.0], [-0.4, 8.0, 0.3], [0.1, 0.5, 8.5]])


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ew.load()


def points(n, spread, seed):
    rng = np.random.default_rng([53, n, seed])
    p = rng.uniform(-1, 2, (n, 3)) @ LAT
    near = 0.02 * rng.uniform(0, 1, (n, 3)) @ LAT
    if spread == "brick":
        p = near
    elif spread == "half":
        p[::2] = near[::2]
    else:
        p[:3] = [[0, 0, 0], LAT[0], -1e-17 * np.ones(3)]  # faces of the cell
    return torch.tensor(p, device="cuda")


def coefficients(grid, orbitals):
    return torch.rand(grid + (orbitals,), dtype=torch.float64, device="cuda",
                      generator=torch.Generator("cuda").manual_seed(3))


def outputs(n, orbitals, der):
    f = dict(dtype=torch.float64, device="cuda")
    return [torch.full((n, orbitals), 7.0, **f)] + (
        [torch.full((n, 3, orbitals), 7.0, **f), torch.full((n, orbitals), 7.0, **f)] if der else [])


# grid, orbitals, points: the smallest numbers of points in the range, whole and cut
# workgroups of the sort, odd and even orbital counts around the slices (64 and 128)
@pytest.mark.parametrize("grid,orbitals,n", [((41, 39, 43), 48, 20400), ((41, 39, 43), 64, 15360), ((13, 40, 40), 127, 8193),
                                             ((24, 24, 24), 260, 4001), ((16, 18, 19), 513, 2048)])
@pytest.mark.parametrize("spread", ["cell", "brick", "half"])
@pytest.mark.parametrize("der", [True, False])
def test_sorted_equals_unsorted(grid, orbitals, n, spread, der):
    coef, p = coefficients(grid, orbitals), points(n, spread, orbitals)
    assert coef.numel() * 8 > 16e6 and orbitals >= 48 and n >= 2048 and 512.0 * n * orbitals >= 0.5e9 and n >= coef[..., 0].numel() / 16
    b = ew.Blips(LAT, grid, orbitals)
    one, many = outputs(n, orbitals, der), outputs(n, orbitals, der)
    b.eval(coef, p, *one)
    for i in range(0, n, 1000):
        b.eval(coef, p[i:i + 1000], *[x[i:i + 1000] for x in many])
    torch.cuda.synchronize()
    for x, y in zip(one, many):
        assert torch.equal(x, y)


def test_one_brick_is_not_slow():
    grid, orbitals, n = (40, 40, 40), 64, 40000
    coef, out = coefficients(grid, orbitals), outputs(n, orbitals, True)
    b = ew.Blips(LAT, grid, orbitals)
    best = {}
    for spread in ("cell", "brick"):
        p = points(n, spread, 1)
        for _ in range(6):
            e0, e1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            e0.record()
            b.eval(coef, p, *out)
            e1.record()
            torch.cuda.synchronize()
            best[spread] = min(best.get(spread, 1e9), e0.elapsed_time(e1))
    print(f"[blip sort] ms {best}", flush=True)
    assert best["brick"] <= 3 * best["cell"]
