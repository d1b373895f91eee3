"""The work that a quantum Monte Carlo program has this library do.

A program sets up its periodic cell and a batch of walkers once (`prepare`), and
then repeats one of four things (`run`):

* "block": the energies of all walkers, then a sweep of single-particle moves
  whose decisions are known beforehand (`Batch.energy` + `Batch.run_moves`, or
  `Batch.run_moves_grad` where the gradient and Laplacian of the Jastrow factor
  are wanted);
* "steps": the move loop step by step, each step applying the previous move's
  decision and returning the next move's energy change (`Batch.step`, and
  `Batch.accept` for the last);
* "energy": the energies of a population of walkers;
* "blip": orbitals, gradients and Laplacians at a batch of points
  (`Blips.eval`).

The launch shapes are those that the library chooses by itself. Inputs are
drawn like those of the repository's workloads: positions uniform in the cell,
Gaussian displacements of 0.3 bohr, decisions independent of the energy change.
"""
import math

import numpy as np
import torch

from paper_2507_02888_amd import ewald as ew
from paper_2507_02888_amd import workloads as wl

SIGMA = 0.3
F8 = torch.float64


# ---- cases -----------------------------------------------------------------------

def _case(name, kind, cell, n, walkers, moves=0, precision="fp64", rs=1.0, gmul=8.0, accept=0.5, refresh=64,
          jastrow=False, u=False, grad=False):
    return dict(name=name, kind=kind, cell=cell, n=n, walkers=walkers, moves=moves, precision=precision, rs=rs,
                gmul=gmul, accept=accept, refresh=refresh, jastrow=jastrow, u=u, grad=grad)


def _blip_case(name, cell, n, grid, orbitals, points, grad=True):
    return dict(name=name, kind="blip", cell=cell, n=n, rs=1.0, grid1=grid[0], grid2=grid[1], grid3=grid[2],
                orbitals=orbitals, points=points, grad=grad)


def listed():
    return [
        # the smallest call: one walker of a 54-electron gas, one block (latency)
        _case("sc54_one_walker", "block", "sc", 54, 1, 54, accept=1.0),
        # a small population stepped move by move with drift (gradient and Laplacian of the full Jastrow factor)
        _case("sc54_steps_drift_mixed", "steps", "sc", 54, 32, 54, "mixed", jastrow=True, u=True, grad=True),
        # a production population of a 250-electron gas, one block of moves
        _case("fcc250_block_mixed", "block", "fcc", 250, 1024, 256, "mixed", rs=2.0),
        # local energies of a large population, with the Jastrow value
        _case("fcc250_energy", "energy", "fcc", 250, 4096, rs=2.0, jastrow=True),
        # the two-dimensional gas
        _case("hex300_block", "block", "hex", 300, 2048, 512, rs=5.0),
        # supercells of three sizes with ions, for a finite-size extrapolation: an uneven batch
        _case("diamond_block_mixed", "block", "diamond", 512, 4096, 256, "mixed"),
        # the headline workload: 1024 electrons, plane-wave Jastrow term, one sweep
        _case("bcc1024_block_mixed", "block", "bcc", 1024, 8192, 1024, "mixed", gmul=12.0, jastrow=True),
        # the same gas in double precision throughout
        _case("bcc1024_block", "block", "bcc", 1024, 1024, 256, gmul=12.0, jastrow=True),
        # the same gas moved step by step, each decision made on the host's side of the call
        _case("bcc1024_steps_mixed", "steps", "bcc", 1024, 8192, 16, "mixed", gmul=12.0, jastrow=True),
        # drift-diffusion sweep with the full Jastrow factor and its derivatives
        _case("bcc1024_drift", "block", "bcc", 1024, 1024, 128, gmul=12.0, jastrow=True, u=True, grad=True),
        # electron-hole bilayer
        _case("bilayer300_block_mixed", "block", "bilayer", 300, 2048, 512, "mixed", rs=5.0),
        # 512 orbitals at one proposed position per walker and move
        _blip_case("blip512", "bcc", 1024, (40, 40, 40), 512, 65536),
    ]


def _log_int(rng, low, high):
    return int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))


def draw(rng):
    if rng.random() < 0.12:
        grid = [rng.randint(8, 40) for _ in range(3)]
        return {k: v for k, v in _blip_case("", rng.choice(("sc", "fcc", "bcc", "triclinic")), rng.randint(54, 1024), grid,
                                            _log_int(rng, 4, 512), _log_int(rng, 32, 65536),
                                            rng.random() < 0.75).items() if k != "name"}
    cell = rng.choice(("sc", "fcc", "bcc", "triclinic", "hex", "oblique", "bilayer", "diamond"))
    kind = rng.choice(("block", "block", "steps", "energy"))
    two_d = cell in ("hex", "oblique", "bilayer")
    n = 512 if cell == "diamond" else _log_int(rng, 8, 1100)
    if cell == "bilayer":
        n += n & 1
    plain = cell in ("bilayer", "diamond")
    jastrow = not plain and rng.random() < 0.5
    u = not plain and rng.random() < 0.3
    moves = {"block": _log_int(rng, 16, 512), "steps": _log_int(rng, 2, 64), "energy": 0}[kind]
    c = _case("", kind, cell, n, _log_int(rng, 1, 8192), moves, rng.choice(("fp64", "mixed")),
              rs=round(rng.uniform(1.0, 5.0), 2), gmul=round(rng.uniform(5.0, 16.0 if two_d else 11.0), 2),
              accept=round(rng.uniform(0.3, 1.0), 2), refresh=rng.choice((16, 64, 64, 256)), jastrow=jastrow, u=u,
              grad=(jastrow or u) and kind != "energy" and rng.random() < 0.5)
    del c["name"]
    while work(c)["flops"] > 2e11 and c["walkers"] > 1:  # a fraction of the largest listed case
        c["walkers"] = c["walkers"] * 2 // 3
    return c


# ---- systems ---------------------------------------------------------------------

def _lattice(cell, measure):
    if cell == "triclinic":
        m = np.array([[1.0, 0.0, 0.0], [0.21, 0.97, 0.0], [-0.13, 0.18, 1.05]])
        return m * (measure / abs(np.linalg.det(m))) ** (1.0 / 3.0)
    if cell == "oblique":
        m = np.array([[1.0, 0.0, 0.0], [0.31, 0.93, 0.0], [0.0, 0.0, 1.0]])
        m[:2, :2] *= math.sqrt(measure / abs(np.linalg.det(m[:2, :2])))
        return m
    return {"sc": wl.sc_cell, "fcc": wl.fcc_cell, "bcc": wl.bcc_cell, "hex": wl.hex_cell,
            "bilayer": wl.hex_cell}[cell](measure)


def _inscribed(lat, dim):
    """Half the shortest lattice vector."""
    r = np.arange(-3, 4)
    n = np.stack(np.meshgrid(*[r] * dim, indexing="ij"), -1).reshape(-1, dim)
    d = np.linalg.norm(n @ lat[:dim, :dim], axis=1)
    return 0.5 * float(d[d > 1e-9].min())


def _systems(case):
    """The cells of a case and how many walkers each has (workloads.System, count)."""
    W, cell, n = case["walkers"], case["cell"], case["n"]
    if cell == "diamond":  # 2^3, 3^3 and 4^3 supercells: 64, 216 and 512 electrons
        counts = [W - 2 * (W // 3), W // 3, W // 3]
        return [(wl.diamond_supercell(k), c) for k, c in zip((2, 3, 4), counts) if c > 0]
    dim = 2 if cell in ("hex", "oblique", "bilayer") else 3
    rs = case["rs"]
    measure = math.pi * rs * rs * n if dim == 2 else 4.0 / 3.0 * math.pi * rs ** 3 * n
    lat = _lattice(cell, measure)
    L = measure ** (1.0 / dim)
    r_ins = _inscribed(lat, dim)
    s = wl.System(name=f"{cell}{n}", dim=dim, lattice=lat, n_mobile=n, mobile_q=-np.ones(n),
                  fixed_pos=np.zeros((0, dim)), fixed_q=np.zeros(0), alpha=5.0 / L, r_cut=min(0.5 * L, 0.999 * r_ins),
                  g_cut=case["gmul"] * 2.0 * math.pi / L)
    if cell == "bilayer":
        h = n // 2
        s.mobile_q = np.concatenate([-np.ones(h), np.ones(n - h)])
        s.mobile_layer = np.concatenate([np.zeros(h, dtype=np.int32), np.ones(n - h, dtype=np.int32)])
        s.layer_z = np.array([0.0, rs])
        s.fixed_layer = np.zeros(0, dtype=np.int32)
    if case["u"]:  # Kato cusp at zero, order C = 3 at the cutoff, seeded coefficients between
        Lu = 0.999 * r_ins
        a = np.random.default_rng(5).uniform(-0.5, 0.5, (2, wl.U_TERMS)) / Lu ** (np.arange(wl.U_TERMS) + wl.U_C)
        for c in (0, 1):
            g = wl.cusp_slope(dim, c == 0)
            a[c, 1] = (g - wl.U_C * a[c, 0] * (-Lu) ** (wl.U_C - 1)) / (-Lu) ** wl.U_C
        s.u_alpha, s.u_C, s.u_cut = a, wl.U_C, Lu
        s.mobile_spin = (np.arange(n) >= n // 2).astype(np.int32)
    return [(s, W)]


def _jastrow_a(case):
    return np.random.default_rng(4).uniform(-0.01, 0.01, 2048) if case["jastrow"] else None


def _inputs(case, seed, device):
    """Packed positions [total][dim], moves k [S][W], proposals [S][W][dim] and decisions [S][W]."""
    g = torch.Generator(device=device).manual_seed(int(seed))
    groups, S = _systems(case), case["moves"]
    pos, ks, news, accs = [], [], [], []
    for s, W in groups:
        d, N = s.dim, s.n_mobile
        lat = torch.tensor(s.lattice[:d, :d], dtype=F8, device=device)
        cur = torch.rand((W, N, d), generator=g, dtype=F8, device=device) @ lat
        pos.append(cur.reshape(W * N, d).clone())
        acc = torch.rand((S, W), generator=g, dtype=F8, device=device) < case["accept"]
        new = SIGMA * torch.randn((S, W, d), generator=g, dtype=F8, device=device)
        for m0 in range(0, S, N):  # electron m mod N moves at step m
            c = min(N, S - m0)
            new[m0:m0 + c] += cur[:, :c].transpose(0, 1)
            a = acc[m0:m0 + c].T[..., None]
            cur[:, :c] = torch.where(a, new[m0:m0 + c].transpose(0, 1), cur[:, :c])
        ks.append((torch.arange(S, device=device, dtype=torch.int32) % N)[:, None].expand(S, W))
        news.append(new)
        accs.append(acc.to(torch.uint8))
    return (torch.cat(pos), torch.cat(ks, 1).contiguous(), torch.cat(news, 1).contiguous(),
            torch.cat(accs, 1).contiguous())


def _blip_inputs(case, seed, device):
    g = torch.Generator(device=device).manual_seed(int(seed))
    grid = (case["grid1"], case["grid2"], case["grid3"])
    lat = _lattice(case["cell"], 4.0 / 3.0 * math.pi * case["rs"] ** 3 * case["n"])
    coef = 2.0 * torch.rand(grid + (case["orbitals"],), generator=g, dtype=F8, device=device) - 1.0
    pts = torch.rand((case["points"], 3), generator=g, dtype=F8, device=device)
    pts = pts @ torch.tensor(lat, dtype=F8, device=device)
    pts += SIGMA * torch.randn((case["points"], 3), generator=g, dtype=F8, device=device)
    return lat, grid, coef, pts


# ---- one pass --------------------------------------------------------------------

def prepare(case, seed):
    dev = "cuda"
    if case["kind"] == "blip":
        lat, grid, coef, pts = _blip_inputs(case, seed, dev)
        P, M = case["points"], case["orbitals"]
        out = dict(val=torch.zeros((P, M), dtype=F8, device=dev))
        if case["grad"]:
            out["grad"] = torch.zeros((P, 3, M), dtype=F8, device=dev)
            out["lap"] = torch.zeros((P, M), dtype=F8, device=dev)
        return dict(case=case, blips=ew.Blips(lat, grid, M), coef=coef, pts=pts, out=out)
    pos, k, new, acc = _inputs(case, seed, dev)
    mixed = case["precision"] == "mixed"
    groups = _systems(case)
    handles = [ew.System(s, precision=ew.EWALD_FP32_MIXED if mixed else ew.EWALD_FP64,
                         refresh_every=case["refresh"] if mixed else 0, jastrow_a=_jastrow_a(case)) for s, _ in groups]
    which = np.concatenate([np.full(W, i, dtype=np.int32) for i, (_, W) in enumerate(groups)])
    batch = ew.Batch(handles, which, device=dev)
    W, S, dim = batch.n_walkers, case["moves"], batch.dim
    jas = case["jastrow"] or case["u"]
    st = dict(case=case, batch=batch, pos=pos, k=k, new=new, acc=acc, out={},
              energy=torch.zeros(W, dtype=F8, device=dev),
              jastrow=torch.zeros(W, dtype=F8, device=dev) if jas else None, delta=None, dj=None, grad=None, lap=None)
    out = st["out"]
    if case["kind"] != "steps":
        out["energy"] = st["energy"]
        if jas:
            out["jastrow"] = st["jastrow"]
    if S:
        out["delta"] = st["delta"] = torch.zeros((S, W), dtype=F8, device=dev)
        if jas:
            out["djastrow"] = st["dj"] = torch.zeros((S, W), dtype=F8, device=dev)
        if case["grad"]:
            out["jgrad"] = st["grad"] = torch.zeros((S, W, dim), dtype=F8, device=dev)
            out["jlap"] = st["lap"] = torch.zeros((S, W), dtype=F8, device=dev)
    # the walkers' state as the header describes it: counters, positions, structure factor
    w = 0
    for h, (s, Wg) in zip(handles, groups):
        b0, p0, r0 = ew.ewald_state_offsets(batch.handle, w)
        size = (batch.state_bytes if w + Wg == W else ew.ewald_state_offsets(batch.handle, w + Wg)[0]) - b0
        rows = batch.state[b0:b0 + size].view(Wg, size // Wg)
        planes = 2 if s.layer_z is not None else 1
        out["counters_%d" % s.n_mobile] = rows[:, :16].view(torch.int32)
        out["positions_%d" % s.n_mobile] = rows[:, p0 - b0:p0 - b0 + s.n_mobile * dim * 8].view(F8)
        out["rho_%d" % s.n_mobile] = rows[:, r0 - b0:r0 - b0 + 16 * planes * h.info["n_slots"]].view(F8)
        w += Wg
    if case["kind"] == "steps":
        batch.energy(pos, st["energy"], st["jastrow"])
    return st


def run(st):
    case = st["case"]
    if case["kind"] == "blip":
        out = st["out"]
        st["blips"].eval(st["coef"], st["pts"], out["val"], out.get("grad"), out.get("lap"))
        return out
    b, k, new, acc, delta, dj, grad, lap = (st[x] for x in ("batch", "k", "new", "acc", "delta", "dj", "grad", "lap"))
    if case["kind"] == "steps":
        for m in range(case["moves"]):
            b.step(acc[m - 1] if m else None, k[m], new[m], delta[m], None if dj is None else dj[m],
                   None if grad is None else grad[m], None if lap is None else lap[m])
        b.accept(acc[case["moves"] - 1])
        return st["out"]
    b.energy(st["pos"], st["energy"], st["jastrow"])
    if case["kind"] == "block":
        if grad is None:
            b.run_moves(k, new, acc, delta, dj)
        else:
            b.run_moves_grad(k, new, acc, delta, dj, grad, lap)
    return st["out"]


# ---- what a pass cannot do without -------------------------------------------------

def _g_count(s):
    """|H|, from the ball's volume."""
    vol = math.pi * s.g_cut ** 2 if s.dim == 2 else 4.0 / 3.0 * math.pi * s.g_cut ** 3
    return max(1.0, 0.5 * vol * s.measure / (2.0 * math.pi) ** s.dim)


def work(case):
    if case["kind"] == "blip":
        P, M = case["points"], case["orbitals"]
        rows = case["grid1"] * case["grid2"] * case["grid3"]
        outs = 5 if case["grad"] else 1
        return dict(bytes=8.0 * (min(rows, 64 * P) * M + 3 * P + outs * P * M), flops=2.0 * outs * 64 * P * M)
    S, total_b, total_f = case["moves"], 0.0, 0.0
    for s, W in _systems(case):
        N, F, G = s.n_mobile, s.n_fixed, _g_count(s)
        state = 16.0 * G + 8.0 * s.dim * N
        pair = 55.0 + (22.0 if case["u"] else 0.0)
        recip = 36.0 + (16.0 if case["grad"] else 0.0)
        per_move_b = 8.0 * s.dim + 5 + 8.0 * (1 + (1 if case["jastrow"] or case["u"] else 0)
                                              + ((s.dim + 1) if case["grad"] else 0))
        per_move_f = G * recip + 2.0 * (N + F - 1) * pair
        energy_f = 10.0 * N * G + (0.5 * N * (N - 1) + N * F) * pair
        if case["kind"] != "steps":
            total_b += W * (8.0 * s.dim * N + state + 16)
            total_f += W * energy_f
        if case["kind"] == "steps":  # rho and positions read once a step, rho written where a move is accepted
            total_b += W * S * (state + 16.0 * G * case["accept"])
        if S:
            total_b += W * (S * per_move_b + state)
            total_f += W * S * per_move_f
            if case["precision"] == "mixed" and case["refresh"]:
                total_f += W * (S * case["accept"] // case["refresh"]) * 10.0 * N * G
    return dict(bytes=total_b, flops=total_f)


# ---- the same in plain 64-bit torch --------------------------------------------------

def _slots(s):
    """Reduced coordinates, |G|^2 and validity of the structure factor's entries: the half set in columns of
    equal leading coordinates, each cut into runs of four (the last run continued past the cutoff), entry j of
    run i at j * runs + i."""
    d = s.dim
    B = 2.0 * math.pi * np.linalg.inv(s.lattice[:d, :d]).T
    nb = [int(math.ceil(s.g_cut * np.linalg.norm(s.lattice[i, :d]) / (2 * math.pi))) for i in range(d)]
    n = np.stack(np.meshgrid(*[np.arange(-b, b + 1) for b in nb], indexing="ij"), -1).reshape(-1, d)
    g2 = ((n @ B) ** 2).sum(1)
    first = np.zeros(len(n), dtype=int)
    for i in range(d - 1, -1, -1):
        first = np.where(n[:, i] != 0, n[:, i], first)
    n = n[(first > 0) & (g2 <= s.g_cut ** 2 * (1 + 1e-12))]
    runs, i = [], 0
    while i < len(n):
        j = i
        while j < len(n) and (n[j, :-1] == n[i, :-1]).all():
            j += 1
        runs += [(n[t], min(4, j - t)) for t in range(i, j, 4)]
        i = j
    step = np.zeros(d, dtype=int)
    step[-1] = 1
    n = np.stack([r + j * step for j in range(4) for r, _ in runs])
    valid = np.array([j < c for j in range(4) for _, c in runs])
    return n, ((n @ B) ** 2).sum(1), valid, B


class _Exact:
    """Energies, Jastrow values and their changes for a group of walkers at once."""

    def __init__(self, case, s, dev):
        self.s, self.dev, self.d = s, dev, s.dim
        d = s.dim
        t = lambda x: torch.tensor(np.asarray(x), dtype=F8, device=dev)  # noqa: E731
        n, g2, valid, B = _slots(s)
        self.n, self.g2, self.lat = t(n), t(g2), t(s.lattice[:d, :d])
        self.G = t(n @ B)
        g = np.sqrt(g2)
        a, om = s.alpha, s.measure
        from scipy.special import erf, erfc, erfcx
        w = 4 * math.pi / om * np.exp(-g2 / (4 * a * a)) / g2 if d == 3 else 2 * math.pi / om * erfc(g / (2 * a)) / g
        self.w = t(np.where(valid, w, 0.0))
        self.q = t(s.mobile_q)
        self.fq, self.fpos = t(s.fixed_q), t(s.fixed_pos)
        self.dz2, self.layer, self.wx = 0.0, None, None
        q2 = float((s.mobile_q ** 2).sum() + (s.fixed_q ** 2).sum())
        qt = float(s.mobile_q.sum() + s.fixed_q.sum())
        self.const = -a / math.sqrt(math.pi) * q2
        if s.layer_z is not None:
            z = float(s.layer_z[1] - s.layer_z[0])
            self.dz2, self.layer = z * z, torch.tensor(s.mobile_layer, device=dev)
            z = abs(z)
            up = np.exp(z * g - (g / (2 * a) + z * a) ** 2) * erfcx(g / (2 * a) + z * a)
            self.wx = t(np.where(valid, math.pi / om * (up + np.exp(-z * g) * erfc(g / (2 * a) - z * a)) / g, 0.0))
            Q = [float(s.mobile_q[np.asarray(s.mobile_layer) == i].sum()) for i in (0, 1)]
            c = lambda x: -2 * math.pi / om * (x * erf(x * a) + math.exp(-(a * x) ** 2) / (a * math.sqrt(math.pi)))  # noqa: E731
            self.const += 0.5 * (Q[0] ** 2 + Q[1] ** 2) * c(0.0) + Q[0] * Q[1] * c(z)
        elif d == 3:
            self.const -= math.pi / (2 * om * a * a) * qt * qt
        else:
            self.const -= math.sqrt(math.pi) / (om * a) * qt * qt
        self.a = None
        if case["jastrow"]:
            order = np.argsort(g2, kind="stable")
            shell, last, idx = np.zeros(len(g2), dtype=int), -1.0, -1
            for o in order:
                if not valid[o]:
                    continue
                if last < 0 or g2[o] > last * (1 + 1e-9):
                    last, idx = g2[o], idx + 1
                shell[o] = idx
            self.a = t(np.where(valid, _jastrow_a(case)[shell], 0.0))
        self.spin = None if s.u_alpha is None else torch.tensor(s.mobile_spin, device=dev)
        sh = np.stack(np.meshgrid(*[np.arange(-1, 2)] * d, indexing="ij"), -1).reshape(-1, d)
        self.shifts = t(sh @ s.lattice[:d, :d])
        if s.n_fixed:
            rf = self.disp(self.fpos[:, None, :], self.fpos[None, :, :])[1].sqrt()
            term = torch.where((rf < s.r_cut) & (rf > 0), self.phi(rf.clamp(min=1e-3)), torch.zeros_like(rf))
            self.const += 0.5 * float((term * self.fq[:, None] * self.fq[None, :]).sum())

    def phi(self, r):
        return torch.erfc(self.s.alpha * r) / r

    def disp(self, a, b):
        """Minimum-image displacement a - b and its square."""
        f = (a - b) @ torch.linalg.inv(self.lat)
        r0 = (f - f.round()) @ self.lat
        best, r2 = r0, (r0 * r0).sum(-1)
        for v in self.shifts:
            c = r0 + v
            c2 = (c * c).sum(-1)
            best = torch.where((c2 < r2)[..., None], c, best)
            r2 = torch.minimum(r2, c2)
        return best, r2

    def u_of(self, r, unequal):
        """u(r), u'(r), u''(r)."""
        s = self.s
        tot = []
        C, L = s.u_C, s.u_cut
        x = r - L
        for ch in (0, 1):
            p = [torch.zeros_like(r) for _ in range(3)]
            for c in s.u_alpha[ch][::-1]:
                p[2] = p[2] * r + 2 * p[1]
                p[1] = p[1] * r + p[0]
                p[0] = p[0] * r + float(c)
            f, f1, f2 = x ** C, C * x ** (C - 1), C * (C - 1) * x ** max(C - 2, 0)
            tot.append((p[0] * f, p[1] * f + p[0] * f1, p[2] * f + 2 * p[1] * f1 + p[0] * f2))
        ins = r < L
        return [torch.where(ins, torch.where(unequal, tot[1][i], tot[0][i]), torch.zeros_like(r)) for i in range(3)]

    def phases(self, r):
        """exp(iG.r) for positions [..., d], as [..., slots] complex."""
        f = r @ torch.linalg.inv(self.lat)
        x = (f - f.floor()) @ self.n.T
        x = (x - x.round()) * (2 * math.pi)
        return torch.complex(x.cos(), x.sin())

    def rho(self, pos):
        """[planes][W][slots]."""
        W, N, _ = pos.shape
        out = torch.zeros((2 if self.layer is not None else 1, W, len(self.w)), dtype=torch.complex128, device=self.dev)
        for i in range(N):
            out[int(self.layer[i]) if self.layer is not None else 0] += self.q[i] * self.phases(pos[:, i])
        for i in range(len(self.fq)):
            out[0] += self.fq[i] * self.phases(self.fpos[i])
        return out

    def energy(self, pos, rho):
        W, N, _ = pos.shape
        e = ((rho.abs() ** 2) @ self.w).sum(0)
        if self.wx is not None:
            e += 2 * (rho[0] * rho[1].conj()).real @ self.wx
        j = (rho[0].abs() ** 2) @ self.a if self.a is not None else torch.zeros(W, dtype=F8, device=self.dev)
        for i in range(N):
            if i + 1 < N:
                r2 = self.disp(pos[:, i, None], pos[:, i + 1:])[1]
                if self.layer is not None:
                    r2 = r2 + self.dz2 * (self.layer[i + 1:] != self.layer[i])
                r = r2.sqrt()
                t = torch.where(r < self.s.r_cut, self.phi(r), torch.zeros_like(r))
                e += self.q[i] * (t @ self.q[i + 1:])
                if self.spin is not None:
                    j += self.u_of(r, (self.spin[i + 1:] != self.spin[i]).expand_as(r))[0].sum(-1)
            if len(self.fq):
                r = self.disp(pos[:, i, None], self.fpos[None])[1].sqrt()
                e += self.q[i] * (torch.where(r < self.s.r_cut, self.phi(r), torch.zeros_like(r)) @ self.fq)
        return e + self.const, j

    def move(self, pos, rho, k, new, acc, want_grad):
        """Change of energy and Jastrow value of moving particle k, then the move where accepted."""
        W, N, d = pos.shape
        s, q = self.s, float(self.q[k])
        old = pos[:, k].clone()
        lk = int(self.layer[k]) if self.layer is not None else 0
        en = self.phases(new)
        delta = q * (en - self.phases(old))
        t = 2 * (rho[lk].conj() * delta).real + delta.abs() ** 2
        dE = t @ self.w
        if self.wx is not None:
            dE += 2 * (rho[1 - lk].conj() * delta).real @ self.wx
        dJ = t @ self.a if self.a is not None else torch.zeros_like(dE)
        others = torch.arange(N, device=self.dev) != k
        keep = []
        for r0 in (new, old):
            x, r2 = self.disp(r0[:, None], pos)
            if self.layer is not None:
                r2 = r2 + self.dz2 * (self.layer != lk)
            r = torch.where(others, r2, torch.full_like(r2, 1e8)).sqrt()
            sg = 1.0 if r0 is new else -1.0
            dE += sg * q * (torch.where(r < s.r_cut, self.phi(r), torch.zeros_like(r)) @ self.q)
            if len(self.fq):
                rf = self.disp(r0[:, None], self.fpos[None])[1].sqrt()
                dE += sg * q * (torch.where(rf < s.r_cut, self.phi(rf), torch.zeros_like(rf)) @ self.fq)
            if self.spin is not None:
                uv = self.u_of(r, (self.spin != self.spin[k]).expand_as(r))
                dJ += sg * uv[0].sum(-1)
                keep.append((x, r, uv))
        grad = torch.zeros((W, d), dtype=F8, device=self.dev)
        lap = torch.zeros(W, dtype=F8, device=self.dev)
        if want_grad:
            if self.a is not None:
                z = (rho[0] + delta).conj() * en
                grad = -2 * q * ((z.imag * self.a) @ self.G)
                lap = -2 * q * ((z.real - q) @ (self.a * self.g2))
            if self.spin is not None:
                x, r, uv = keep[0]
                ur = uv[1] / r
                grad = grad + (ur[..., None] * x).sum(1)
                lap = lap + (uv[2] + (d - 1) * ur).sum(-1)
        rho[lk] += torch.where(acc[:, None], delta, torch.zeros_like(delta))
        pos[:, k] = torch.where(acc[:, None], new, old)
        return dE, dJ, grad, lap


def _exact_blip(case, seed, dev):
    lat, grid, coef, pts = _blip_inputs(case, seed, dev)
    P, M = case["points"], case["orbitals"]
    A = torch.tensor(lat, dtype=F8, device=dev)
    n = torch.tensor(grid, dtype=F8, device=dev)
    J = torch.linalg.inv(A) * n  # d x_d / d r_e at [e][d]
    flat = coef.reshape(-1, M)
    out = dict(val=torch.empty((P, M), dtype=F8, device=dev))
    if case["grad"]:
        out.update(grad=torch.empty((P, 3, M), dtype=F8, device=dev), lap=torch.empty((P, M), dtype=F8, device=dev))
    for p0 in range(0, P, 1024):
        x = pts[p0:p0 + 1024] @ torch.linalg.inv(A)
        x = (x - x.floor()) * n
        base = x.floor()
        f = []
        for d in range(3):
            g = base[:, d, None] + torch.arange(-1, 3, device=dev, dtype=F8)
            y = x[:, d, None] - g
            ay, sg = y.abs(), torch.sign(y)
            t = 2 - ay
            inn = ay <= 1
            f.append((torch.where(inn, 1 - 1.5 * y * y + 0.75 * ay ** 3, 0.25 * t ** 3),
                      torch.where(inn, -3 * y + 2.25 * sg * y * y, -0.75 * sg * t * t),
                      torch.where(inn, -3 + 4.5 * ay, 1.5 * t), torch.remainder(g, n[d]).long()))
        idx = (f[0][3][:, :, None, None] * grid[1] + f[1][3][:, None, :, None]) * grid[2] + f[2][3][:, None, None, :]
        rows = flat[idx.reshape(-1)].reshape(len(x), 64, M)
        wt = lambda a, b, c: (f[0][a][:, :, None, None] * f[1][b][:, None, :, None] * f[2][c][:, None, None, :]).reshape(len(x), 64)  # noqa: E731
        ws = [wt(0, 0, 0)]
        if case["grad"]:
            d1 = [wt(1, 0, 0), wt(0, 1, 0), wt(0, 0, 1)]
            ws += [sum(J[e, d] * d1[d] for d in range(3)) for e in range(3)]
            Mx = J.T @ J
            h = {(0, 0): wt(2, 0, 0), (1, 1): wt(0, 2, 0), (2, 2): wt(0, 0, 2), (0, 1): wt(1, 1, 0), (0, 2): wt(1, 0, 1),
                 (1, 2): wt(0, 1, 1)}
            ws.append(sum((1 if a == b else 2) * Mx[a, b] * v for (a, b), v in h.items()))
        got = [(w[:, :, None] * rows).sum(1) for w in ws]
        out["val"][p0:p0 + 1024] = got[0]
        if case["grad"]:
            out["grad"][p0:p0 + 1024] = torch.stack(got[1:4], 1)
            out["lap"][p0:p0 + 1024] = got[4]
    return out


def exact(case, seed):
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    if case["kind"] == "blip":
        return _exact_blip(case, seed, dev)
    S, cost = case["moves"], 0.0
    for s, W in _systems(case):
        im, N, G = 3 ** s.dim + 1, s.n_mobile + s.n_fixed, 1.3 * _g_count(s)
        cost += W * (0.5 * N * N * im + 2 * N * G + S * (2 * N * im + 4 * G))
    if cost > (1e11 if dev == "cuda" else 1e9):
        return None
    pos, k, new, acc = _inputs(case, seed, dev)
    jas = case["jastrow"] or case["u"]
    out = {x: [] for x in ("energy", "jastrow", "delta", "djastrow", "jgrad", "jlap")}
    states, w, row = {}, 0, 0
    for s, W in _systems(case):
        X = _Exact(case, s, dev)
        parts, size = [], max(1, int(2e8 // (s.n_mobile * 3 ** s.dim * 8 + len(X.w) * 16)))
        for w0 in range(w, w + W, size):
            Wc = min(size, w + W - w0)
            p = pos[row:row + Wc * s.n_mobile].reshape(Wc, s.n_mobile, s.dim).clone()
            row += Wc * s.n_mobile
            rho = X.rho(p)
            e, j = X.energy(p, rho) if case["kind"] != "steps" else (None, None)
            moves = [X.move(p, rho, m % s.n_mobile, new[m, w0:w0 + Wc], acc[m, w0:w0 + Wc] != 0, case["grad"])
                     for m in range(S)]
            f = p @ torch.linalg.inv(X.lat)
            rho = X.rho(p).transpose(0, 1).reshape(Wc, -1)
            parts.append((e, j, [torch.stack(x) for x in zip(*moves)] if S else [], (f - f.floor()).reshape(Wc, -1),
                          torch.view_as_real(rho).reshape(Wc, -1)))
        w += W
        states["positions_%d" % s.n_mobile] = torch.cat([x[3] for x in parts])
        states["rho_%d" % s.n_mobile] = torch.cat([x[4] for x in parts])
        for x in parts:
            out["energy"].append(x[0])
            out["jastrow"].append(x[1])
            for name, v in zip(("delta", "djastrow", "jgrad", "jlap"), x[2]):
                out[name].append(v)
    got = {}
    if case["kind"] != "steps":
        got["energy"] = torch.cat(out["energy"])
        if jas:
            got["jastrow"] = torch.cat(out["jastrow"])
    if S:
        got["delta"] = torch.cat(out["delta"], 1)
        if jas:
            got["djastrow"] = torch.cat(out["djastrow"], 1)
        if case["grad"]:
            got["jgrad"], got["jlap"] = torch.cat(out["jgrad"], 1), torch.cat(out["jlap"], 1)
    got.update(states)
    return got
