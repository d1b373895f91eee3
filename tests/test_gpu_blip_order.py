"""Large blip batches, which are served in the order of the points' places on
the grid, against the same points in small calls, which are not: each point's
arithmetic is the same, so every output is bit for bit the same."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2507_02888_amd import ewald as ew

pytestmark = pytest.mark.gpu

SMALL = 1000  # points per call, below the ordered range


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ew.load()


# grid, orbitals, points: coefficient sets just above 16 MB and larger, odd
# and even orbital counts around the slice widths (64, 128 and 256), odd grid
# sides (a brick that is cut short), the smallest ordered batch
@pytest.mark.parametrize("grid,orbitals,points", [((41, 39, 43), 31, 4320), ((41, 39, 43), 64, 4999), ((16, 18, 19), 513, 2048),
                                                  ((13, 40, 40), 129, 3001), ((30, 30, 30), 260, 2500)])
@pytest.mark.parametrize("spread", ["cell", "cluster"])
@pytest.mark.parametrize("der", [True, False])
def test_ordered_equals_unordered(grid, orbitals, points, spread, der):
    rng = np.random.default_rng([41, orbitals, points])
    lat = np.array([[9.0, 0.2, 0.0], [-0.4, 8.0, 0.3], [0.1, 0.5, 8.5]])
    if spread == "cell":
        pts = rng.uniform(-1, 2, (points, 3)) @ lat
        pts[:3] = [[0, 0, 0], lat[0], -1e-17 * np.ones(3)]  # faces of the cell
    else:  # every point in one brick
        pts = 0.02 * rng.uniform(0, 1, (points, 3)) @ lat
    dev = "cuda"
    coef = torch.rand(grid + (orbitals,), dtype=torch.float64, device=dev, generator=torch.Generator(dev).manual_seed(3))
    assert coef.numel() * 8 > 16e6 and points >= 2048 and points >= coef[..., 0].numel() / 16
    p = torch.tensor(pts, device=dev)
    b = ew.Blips(lat, grid, orbitals)

    def outputs():
        f = dict(dtype=torch.float64, device=dev)
        return [torch.full((points, orbitals), 7.0, **f)] + (
            [torch.full((points, 3, orbitals), 7.0, **f), torch.full((points, orbitals), 7.0, **f)] if der else [])

    one, many = outputs(), outputs()
    b.eval(coef, p, *one)
    for i in range(0, points, SMALL):
        b.eval(coef, p[i:i + SMALL], *[x[i:i + SMALL] for x in many])
    torch.cuda.synchronize()
    for x, y in zip(one, many):
        assert torch.equal(x, y)
