"""The fused sweep's launch shapes when nothing is fixed (chosen by the walkers
per compute unit) against the shapes fixed by hand, at the walker counts where
the choice changes; and the staging of chunks against the per-step calls, on
sequences that move few particles again and again, with chunks of 1, 2, 63 and
64 moves.

Tolerances, from before any run: shapes that differ in the waves per SIMD only,
or in the order of FP64 sums, agree to rounding: N_terms roundings of terms that
are below the total energy or the largest change of it, 1e-12 of it (at most 1024 particles and 990 segments
of 8 terms: 10^4 roundings of 1.1e-16).  512 x 2 and 1024 x 1 in the mixed form
add the same FP32 segment sums and the same FP32 pair terms up in FP64, so the same bound
holds.  The fused sweep against the per-step calls in the mixed form: FP32
partial sums over other groups, 1e-6 Ha and 3e-6 on Jastrow deltas.
"""
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


def cus():
    return torch.cuda.get_device_properties(0).multi_processor_count


class Sweep:
    """W walkers of one seeded system, and S moves of particles below `among`."""

    def __init__(self, cfg_id, W, S, precision, u_term=False, among=None, K=3):
        s = wl.config(cfg_id).systems[0]
        if u_term:
            s = wl.with_u_term(s, cfg_id)
        self.W, self.S, self.dim, self.n = W, S, s.dim, s.n_mobile
        rng = np.random.default_rng([17, cfg_id, W, S])
        lat = s.lattice[:s.dim, :s.dim]
        self.ja = rng.uniform(-0.01, 0.01, 64)
        self.sys = ew.System(s, precision=precision, refresh_every=K if precision == MIXED else 0, jastrow_a=self.ja)
        self.batch = ew.Batch([self.sys], np.zeros(W, np.int32))
        pos = rng.random((W, s.n_mobile, s.dim)) @ lat
        k = rng.integers(0, among or s.n_mobile, (S, W)).astype(np.int32)
        k[rng.random((S, W)) < 0.05] = -1  # an invalid index: NaN, and no move
        self.k = torch.tensor(k, device="cuda")
        self.new = torch.tensor(rng.random((S, W, s.dim)) @ lat, device="cuda")
        self.acc = torch.tensor(rng.integers(0, 2, (S, W)).astype(np.uint8), device="cuda")
        self.pos = torch.tensor(pos.reshape(-1, s.dim), device="cuda")
        self.e = torch.zeros(W, dtype=torch.float64, device="cuda")
        self.scale = None

    def start(self):
        self.batch.energy(self.pos, self.e, torch.zeros_like(self.e))
        torch.cuda.synchronize()
        self.scale = max(1.0, float(self.e.abs().max()))

    def result(self, der=False):
        """[dE, dJ, (grad, lap)] of the fused sweep and rho of the first and last walkers."""
        self.start()
        o = [torch.zeros((self.S, self.W), dtype=torch.float64, device="cuda") for _ in range(3)]
        if der:
            g = torch.zeros((self.S, self.W, self.dim), dtype=torch.float64, device="cuda")
            self.batch.run_moves_grad(self.k, self.new, self.acc, o[0], o[1], g, o[2])
            outs = [o[0], o[1], g, o[2]]
        else:
            self.batch.run_moves(self.k, self.new, self.acc, o[0], o[1])
            outs = o[:2]
        torch.cuda.synchronize()
        self.scale = max(self.scale, float(torch.nan_to_num(o[0]).abs().max()))
        return [x.cpu().numpy() for x in outs] + [self.batch.walker_rho(w) for w in (0, self.W - 1)]


def check(a, b, tols, what):
    for i, (x, y) in enumerate(zip(a, b)):
        assert np.array_equal(np.isnan(x), np.isnan(y)), (what, i)
        d = float(np.max(np.abs(np.nan_to_num(x - y))))
        print(f"  {what} output {i}: {d:.3e} (allowed {tols[i]:.1e})", flush=True)
        assert d <= tols[i], (what, i, d)


@pytest.mark.parametrize("precision", [FP64, MIXED], ids=["fp64", "mixed"])
@pytest.mark.parametrize("rounds,more,waves", [(0, 1, 2), (2, 0, 2), (2, 1, 3), (3, 1, 4), (4, 1, 3)])
def test_small_walkers_default_waves(precision, rounds, more, waves):
    W = rounds * cus() + more
    s = Sweep(2, W, 6, precision)
    got = s.result()
    t = s.batch.tuning()
    print(f"[waves] W={W} {t}", flush=True)
    assert t["threads"] == 256 and t["waves"] == waves
    s.batch.set_tuning(threads=256, waves=2)
    tol = 1e-12 * s.scale
    check(got, s.result(), [tol, tol, 1e-9, 1e-9], "two waves")


@pytest.mark.parametrize("precision", [FP64, MIXED], ids=["fp64", "mixed"])
@pytest.mark.parametrize("rounds,more,threads", [(1, 0, 1024), (1, 1, 512), (2, 0, 512), (2, 1, 1024)])
def test_large_walkers_default_threads(precision, rounds, more, threads):
    W = rounds * cus() + more
    s = Sweep(5, W, 5, precision)
    got = s.result()
    t = s.batch.tuning()
    print(f"[threads] W={W} {t}", flush=True)
    assert t["threads"] == threads and t["waves"] == (4 if threads == 512 else 0)
    s.batch.set_tuning(threads=1024)
    tol = 1e-12 * s.scale
    check(got, s.result(), [tol, tol, 1e-9, 1e-9], "1024 threads")


@pytest.mark.parametrize("precision", [FP64, MIXED], ids=["fp64", "mixed"])
@pytest.mark.parametrize("u_term", [False, True], ids=["p", "pu"])
def test_derivative_sweep_default(precision, u_term):
    s = Sweep(5, 3, 9, precision, u_term=u_term)
    got = s.result(der=True)
    s.batch.set_tuning(threads=1024)
    ref = s.result(der=True)
    tol = 1e-12 * s.scale
    # derivative sums stay FP32 within a segment in both shapes
    print(f"[derivatives] {u_term}", flush=True)
    check(got, ref, [tol, tol, 1e-11 * max(1.0, float(np.nanmax(np.abs(ref[2])))),
                     1e-11 * max(1.0, float(np.nanmax(np.abs(ref[3])))), 1e-9, 1e-9], "1024 threads")


@pytest.mark.parametrize("precision", [FP64, MIXED], ids=["fp64", "mixed"])
@pytest.mark.parametrize("chunk", [1, 2, 63, 64])
@pytest.mark.parametrize("moves", [1, 65, 130])
def test_chunks_of_repeated_particles(precision, chunk, moves):
    s = Sweep(1, 2, moves, precision, among=3, K=11)
    s.batch.set_tuning(chunk=chunk)
    got = s.result()[:2]
    s.start()
    d = torch.zeros((moves, 2), dtype=torch.float64, device="cuda")
    dj = torch.zeros_like(d)
    for m in range(moves):
        s.batch.move_delta(s.k[m], s.new[m], d[m], dj[m])
        s.batch.accept(s.acc[m])
    torch.cuda.synchronize()
    t = 1e-12 * s.scale * moves if precision == FP64 else 1e-6
    tj = 1e-12 * s.scale * moves if precision == FP64 else 3e-6
    print(f"[chunks] {chunk} of {moves}", flush=True)
    check(got, [d.cpu().numpy(), dj.cpu().numpy()], [t, tj], "per-step calls")
