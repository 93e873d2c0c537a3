"""Performance cases: the work that programs built on this library give it, through its public
entry points, from one step of a 1e4-particle beam to ten steps of a 1e8-particle one.

Every beam is a 6-D Gaussian electron bunch (1 nC, 20 MeV; see `SIGMA`), tracked through thin
or thick FODO lattices.  Programs that evaluate an objective start every evaluation from the
same draws (`init_from_normals`), so most passes do too; long production runs and batches go on
from where the last call ended.  With the float32 grid the particles are handed on as a float32
dump, the precision such a run has.
"""
import math

import torch

import paper_2208_02382_amd as pic
from paper_2208_02382_amd import autotune

MASS_MEV = 0.510998950
QM_QEEV = -1.0e-6 / MASS_MEV
CHARGE_C = 1.0e-9
KIN_MEV = 20.0
SIGMA = (1e-3, 1e-3, 1e-3, 1e-3, 5e-3, 1e-3)   # rms of x, px, y, py, z, delta
THIN, DRIFT, QUAD = 0, 1, 2
# the thick FODO cell (kind, k [1/m^2], ds [m], slices)
THICK_FODO = ((DRIFT, 0.0, 0.25, 25), (QUAD, 1.0, 1.0, 25), (DRIFT, 0.0, 0.5, 25),
              (QUAD, -1.0, 1.0, 25), (DRIFT, 0.0, 0.25, 25))
# the same cell in few slices, so that a short call passes every kind of element
THICK_SHORT = ((DRIFT, 0.0, 0.25, 1), (QUAD, 1.0, 1.0, 3), (DRIFT, 0.0, 0.5, 1),
               (QUAD, -1.0, 1.0, 3), (DRIFT, 0.0, 0.25, 1))
# grid nodes per axis whose padded length 2 n is 2^a 3^b
AXIS = (16, 18, 24, 27, 32, 36, 48, 54, 64, 72, 81, 96, 108, 128)


def _case(name, op, n, nodes, shape, steps, **kw):
    c = {"op": op, "n": int(n), "nx": nodes[0], "ny": nodes[1], "nz": nodes[2], "shape": shape,
         "steps": steps, "fp32": False, "lattice": "thin", "halo": 0.0}
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one step and the beam's statistics: the smallest call of an interactive study, all
        # latency
        _case("one-step-1e4-32c", "track", 10_000, (32, 32, 32), 1, 1),
        # a coarse objective evaluation inside an optimiser: launches and the grid
        _case("track-1e4-32c", "track", 10_000, (32, 32, 32), 1, 20),
        # the ordinary objective evaluation
        _case("track-1e6-64c", "track", 1_000_000, (64, 64, 64), 1, 20),
        # the same with the float32 grid, a ragged grid and quadratic shapes
        _case("track-3e5-ragged-tsc-f32", "track", 300_007, (72, 54, 96), 2, 20, fp32=True),
        # the thick FODO cell with the moments written after every slice
        _case("diag-1e5-thick", "diag", 100_003, (48, 48, 48), 2, 25, lattice="thick"),
        # the field without differencing error
        _case("direct-2e5-tsc", "direct", 200_000, (48, 36, 64), 2, 10, lattice="short"),
        # a program that drives the single steps itself
        _case("calls-1e6-64c-tsc", "calls", 1_000_000, (64, 64, 64), 2, 1),
        # one GPU's share of a 1e8-particle beam split over eight, caller's order
        _case("track-1e7-128c-tsc", "track", 12_500_000, (128, 128, 128), 2, 10, halo=0.1),
        # a long production run: the particles stay in tile order between calls, the program
        # looks at the charge density and the moments
        _case("binned-1e8-128c-tsc", "binned", 100_000_000, (128, 128, 128), 2, 10, halo=0.1),
        # the same with the float32 grid
        _case("binned-1e8-128c-tsc-f32", "binned", 100_000_000, (128, 128, 128), 2, 10,
              halo=0.1, fp32=True),
        # a parameter scan: many beams in one graph
        _case("batch-256", "batch", 1_000_000, (64, 64, 64), 1, 10, beams=256),
        # gradients of the final beam in the quadrupole strengths and the initial beam
        _case("adjoint-1e6-64c", "adjoint", 1_000_000, (64, 64, 64), 1, 20, lattice="quads8",
              ckpt=10),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _nodes(rng, hi):
    ax = [a for a in AXIS if a <= hi]
    if rng.random() < 0.4:
        return (rng.choice(ax),) * 3
    return tuple(rng.choice(ax) for _ in range(3))


def draw(rng):
    op = rng.choice(("track", "track", "track", "binned", "diag", "direct", "calls", "batch",
                     "adjoint"))
    shape = rng.choice((1, 2))
    fp32 = rng.random() < 0.3
    if op in ("track", "binned"):
        n = _log_int(rng, 1e4, 1e8 if op == "binned" else 2e7)
        steps = rng.randint(1, 20)
        if n > 50_000_000:
            steps = min(steps, 10)
        return _case(None, op, n, _nodes(rng, 128), shape, steps, fp32=fp32,
                     lattice=rng.choice(("thin", "thick", "short")),
                     halo=rng.choice((0.0, 0.1)))
    if op == "diag":
        return _case(None, op, _log_int(rng, 1e4, 1e7), _nodes(rng, 128), shape,
                     rng.randint(5, 25), lattice=rng.choice(("thick", "short")))
    if op == "direct":
        return _case(None, op, _log_int(rng, 1e4, 1e7), _nodes(rng, 128), shape,
                     rng.randint(2, 10), fp32=fp32, lattice=rng.choice(("thin", "short")))
    if op == "calls":
        return _case(None, op, _log_int(rng, 1e4, 1e7), _nodes(rng, 128), shape, 1, fp32=fp32)
    if op == "batch":
        return _case(None, op, _log_int(rng, 1e5, 1e6), (64, 64, 64), shape,
                     rng.randint(2, 10), beams=_log_int(rng, 8, 192), fp32=fp32)
    return _case(None, op, _log_int(rng, 1e4, 1e6), _nodes(rng, 64), shape, rng.randint(4, 16),
                 lattice=rng.choice(("quads8", "short")), ckpt=rng.randint(2, 10))


# ------------------------------------------------------------------------------------ inputs

def _lattice(case):
    """(kind, k, ds, slices) elements."""
    if case["lattice"] == "thick":
        return THICK_FODO
    if case["lattice"] == "short":
        return THICK_SHORT
    if case["lattice"] == "quads8":
        return tuple((THIN, 1.0 if i % 2 == 0 else -1.0, 0.5, 1) for i in range(8))
    return ((THIN, 1.0, 0.5, 1), (THIN, -1.0, 0.5, 1))


def _draws(n, halo, seed):
    """Unit normals (6, n), the trailing halo fraction uniform out to 4 sigma."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    xi = torch.randn((6, n), generator=g, dtype=torch.float64, device="cuda")
    nh = int(round(halo * n))
    if nh:
        xi[:, n - nh:].uniform_(-4.0, 4.0, generator=g)
    return xi


def _sigma():
    return torch.diag(torch.tensor(SIGMA, dtype=torch.float64) ** 2)


def _scan(case, seed):
    """The beams of a batch: particle counts, cubic grids and FODO strengths of a scan."""
    g = torch.Generator().manual_seed(seed)
    u = torch.rand((3, case["beams"]), generator=g, dtype=torch.float64)
    lo, hi = math.log(1e4), math.log(float(case["n"]))
    # sizes are the case's, strengths and draws the seed's
    v = torch.rand((2, case["beams"]), generator=torch.Generator().manual_seed(case["beams"]),
                   dtype=torch.float64)
    ns = [int(round(math.exp(lo + (hi - lo) * float(a)))) for a in v[0]]
    gs = [(32, 48, 64)[int(3 * float(a))] for a in v[1]]
    ks = [0.5 + 1.5 * float(a) for a in u[0]]
    return ns, gs, ks


def prepare(case, seed):
    n, shape, fp32 = case["n"], case["shape"], case["fp32"]
    nodes = (case["nx"], case["ny"], case["nz"])
    st = {"op": case["op"], "steps": case["steps"], "fp32": fp32, "sigma": _sigma()}
    if case["op"] == "batch":
        ns, gs, ks = _scan(case, seed)
        flat = torch.empty(6 * sum(ns), dtype=torch.float64, device="cuda")
        beams, at = [], 0
        for b, (nb, gb) in enumerate(zip(ns, gs)):
            X = flat[at:at + 6 * nb].view(6, nb)
            at += 6 * nb
            beam = pic.Beam(nb, QM_QEEV, CHARGE_C, KIN_MEV, MASS_MEV, shape, (gb,) * 3,
                            grid_fp32=fp32, X=X)
            beam.init_from_normals(st["sigma"], _draws(nb, 0.0, seed * 1000 + b))
            beams.append(beam)
        st["batch"] = pic.Batch(beams, [((k, 0.5), (-k, 0.5)) for k in ks])
        st["X"] = flat
        return st
    st["beam"] = pic.Beam(n, QM_QEEV, CHARGE_C, KIN_MEV, MASS_MEV, shape, nodes, grid_fp32=fp32,
                          direct_field=case["op"] == "direct",
                          tuning=autotune.lookup(n, nodes, shape, fp32))
    st["lattice"] = _lattice(case)
    xi = _draws(n, case["halo"], seed)
    if case["op"] == "binned":
        st["beam"].init_from_normals(st["sigma"], xi)
    else:
        st["xi"] = xi
    if case["op"] == "adjoint":
        st["ckpt"] = case["ckpt"]
    return st


def run(st):
    op, steps = st["op"], st["steps"]
    if op == "batch":
        st["batch"].track(steps)
        return st["X"].float() if st["fp32"] else st["X"]
    beam = st["beam"]
    if op == "binned":
        beam.track(st["lattice"], steps, binned=True)
        mom = pic.moments_noalloc(beam.X)
        return {"rho": beam.deposit(), "moments": mom.float() if st["fp32"] else mom}
    beam.init_from_normals(st["sigma"], st["xi"])
    if op == "adjoint":
        m, dk, lam, dL = beam.track_adjoint(st["lattice"], steps, (1.0, 1.0, 1.0, 1.0),
                                            ckpt_every=st["ckpt"], xi=st["xi"])
        return {"m": torch.tensor(m, dtype=torch.float64),
                "dk": torch.tensor(dk, dtype=torch.float64), "lam": lam,
                "dL": torch.tensor(dL, dtype=torch.float64), "X": beam.X}
    if op == "calls":
        beam.push(pic.PUSH_THINQUAD, 1.0)
        beam.push(pic.PUSH_DRIFT, 0.25)
        rho = beam.deposit()
        phi, E = beam.poisson_solve(rho, phi=beam.new_phi())
        Ep = beam.gather(E)
        beam.push(pic.PUSH_KICK, 0.5, Ep)
        beam.push(pic.PUSH_DRIFT, 0.25)
        return {"rho": rho, "phi": phi, "E": E, "Ep": Ep,
                "X": beam.X.float() if st["fp32"] else beam.X}
    if op == "diag":
        d = beam.track(st["lattice"], steps, diagnostics=True)
        return {"diag": d, "X": beam.X}
    beam.track(st["lattice"], steps)
    mom = pic.moments_noalloc(beam.X)
    if st["fp32"]:
        return {"X": beam.X.float(), "moments": mom.float()}
    return {"X": beam.X, "moments": mom}


# -------------------------------------------------------------------------------------- work

def _step_work(n, nodes, shape, es, direct=False):
    """One split-operator step: positions read by the deposit, six coordinates read and written
    by the push; the charge and the field written and read once; a padded forward and inverse
    real transform per convolution and the kernel's spectrum."""
    ng = nodes[0] * nodes[1] * nodes[2]
    nbytes = n * (24 + 96) + 8 * es * ng
    fft = 2.5 * 8 * ng * math.log2(8 * ng)
    ncomp = 3 if direct else 1
    stencil = (shape + 1) ** 3
    flops = n * (stencil * 8 + 60) + fft * (1 + ncomp) + ncomp * (fft / 4 + 100 * ng)
    return nbytes, flops


def work(case):
    es = 4 if case["fp32"] else 8
    n, steps = case["n"], case["steps"]
    nodes = (case["nx"], case["ny"], case["nz"])
    if case["op"] == "batch":
        ns, gs, _ = _scan(case, 0)
        per = [_step_work(a, (g, g, g), case["shape"], es) for a, g in zip(ns, gs)]
        return {"bytes": steps * sum(p[0] for p in per), "flops": steps * sum(p[1] for p in per)}
    b, f = _step_work(n, nodes, case["shape"], es, case["op"] == "direct")
    if case["op"] == "adjoint":
        # forward, and a reverse sweep that reads the state and updates its adjoint
        return {"bytes": steps * 3 * b + 144 * n, "flops": steps * 3 * f}
    if case["op"] == "calls":
        return {"bytes": b + n * (96 + 3 * es) + es * nodes[0] * nodes[1] * nodes[2], "flops": f}
    start = 0 if case["op"] == "binned" else 96 * n
    return {"bytes": steps * b + start + 48 * n, "flops": steps * f}


# ----------------------------------------------------------------------- values in 64 bits

EPS0, CHUNK = 8.8541878128e-12, 20_000_000


def _corner_sum(F):
    for d in range(3):
        F = F.diff(dim=d)
    return F


def _kernels(h, nodes, direct):
    """Cell averages of 1/r (or of u_a/r^3, a = 0, 1, 2) on the octant, [z][y][x]."""
    x, y, z = (torch.cat([torch.zeros(1, dtype=torch.float64, device=h.device),
                          torch.arange(0.5, n + 1, dtype=torch.float64, device=h.device) * ha])
               for ha, n in zip(h, nodes))
    x, y, z = x[None, None, :], y[None, :, None], z[:, None, None]
    r2 = x * x + y * y + z * z
    r = torch.where(r2 == 0, torch.ones_like(r2), r2).sqrt()
    one = torch.ones((), dtype=torch.float64, device=h.device)
    at = [torch.atan2(v * w, torch.where(u == 0, one, u) * r)
          for u, v, w in ((x, y, z), (y, z, x), (z, x, y))]
    Lx, Ly, Lz = ((u + r).log() for u in (x, y, z))
    vol = h[0] * h[1] * h[2]
    if not direct:
        F = (x * y * Lz + y * z * Lx + z * x * Ly
             - 0.5 * (x * x * at[0] + y * y * at[1] + z * z * at[2]))
        out = [_corner_sum(F) / vol]
    else:
        H = (y * Lz + z * Ly - x * at[0], z * Lx + x * Lz - y * at[1],
             x * Ly + y * Lx - z * at[2])
        out = [-_corner_sum(f) / vol for f in H]
    full = []
    for a, G in enumerate(out):
        for d in range(3):   # torch dim d is axis 2 - d
            m = G.shape[d] - 1
            w = torch.ones(m + 1, dtype=torch.float64, device=h.device)
            odd = direct and 2 - d == a
            w[0] = 0.0 if odd else 2.0
            if odd:
                w[m] = 0.0
            G = G * w.reshape([-1 if e == d else 1 for e in range(3)])
            tail = G.narrow(d, 1, m - 1).flip(d)
            G = torch.cat([G, -tail if odd else tail], dim=d)
        full.append(G)
    return full


def _weights(u, shape):
    if shape == 1:
        i = u.detach().floor()
        f = u - i
        return i.long(), (1 - f, f)
    i = (u.detach() + 0.5).floor()
    d = u - i
    return i.long() - 1, (0.5 * (0.5 - d) ** 2, 0.75 - d * d, 0.5 * (0.5 + d) ** 2)


def _stencil(pos, origin, h, nodes, shape):
    ws = [_weights((pos[a] - origin[a]) / h[a], shape) for a in range(3)]
    for c in range(shape + 1):
        for b in range(shape + 1):
            wzy = ws[2][1][c] * ws[1][1][b]
            row = ((ws[2][0] + c) * nodes[1] + ws[1][0] + b) * nodes[0] + ws[0][0]
            for a in range(shape + 1):
                yield row + a, wzy * ws[0][1][a]


def _parts(n):
    return [(i, min(n, i + CHUNK)) for i in range(0, n, CHUNK)]


def _geometry(pos, nodes, gamma):
    lo = torch.stack([p.amin() for p in pos])
    hi = torch.stack([p.amax() for p in pos])
    cells = torch.tensor([m - 3.5 for m in nodes], dtype=torch.float64, device=lo.device)
    h = (hi - lo) / cells
    return lo - 1.25 * h, h, torch.stack([h[0], h[1], gamma * h[2]])


def _deposit(pos, origin, h, nodes, shape, q):
    rho = torch.zeros(nodes[0] * nodes[1] * nodes[2], dtype=torch.float64, device=h.device)
    for i, j in _parts(pos[0].numel()):
        for at, w in _stencil([p[i:j] for p in pos], origin, h, nodes, shape):
            rho = rho.index_add(0, at, q * w) if w.requires_grad else rho.index_add_(0, at, q * w)
    return rho.view(nodes[2], nodes[1], nodes[0])


def _field(rho, hr, nodes, direct):
    """phi on nodes -1..n (None with the direct field) and E' (3, nz, ny, nx)."""
    pad = [2 * nodes[2], 2 * nodes[1], 2 * nodes[0]]
    rk = torch.fft.rfftn(rho, s=pad)
    conv = [torch.fft.irfftn(rk * torch.fft.rfftn(G), s=pad) / (4 * math.pi * EPS0)
            for G in _kernels(hr, nodes, direct)]
    if direct:
        return None, torch.stack([c[:nodes[2], :nodes[1], :nodes[0]] for c in conv])
    phi = conv[0].roll((1, 1, 1), (0, 1, 2))[:nodes[2] + 2, :nodes[1] + 2, :nodes[0] + 2]
    E = torch.stack([(phi[1:-1, 1:-1, :-2] - phi[1:-1, 1:-1, 2:]) / (2 * hr[0]),
                     (phi[1:-1, :-2, 1:-1] - phi[1:-1, 2:, 1:-1]) / (2 * hr[1]),
                     (phi[:-2, 1:-1, 1:-1] - phi[2:, 1:-1, 1:-1]) / (2 * hr[2])])
    return phi, E


def _gather(pos, E, origin, h, nodes, shape):
    flat = E.reshape(3, -1)
    out = []
    for i, j in _parts(pos[0].numel()):
        acc = 0.0
        for at, w in _stencil([p[i:j] for p in pos], origin, h, nodes, shape):
            acc = acc + w * flat[:, at]
        out.append(acc)
    return torch.cat(out, dim=1)


def _half(X, kind, k, s, kq, gamma):
    """Half of a slice: thin quad kq and drift, or the thick element's map over s."""
    x, px, y, py, z, d = X
    if kind == THIN and kq is not None:
        px, py = px - kq * x, py + kq * y
    if kind == QUAD:
        def plane(u, pu, kk):
            w = abs(kk) ** 0.5
            p = w * s
            c, sn = (math.cos(p), math.sin(p)) if kk > 0 else (math.cosh(p), math.sinh(p))
            return c * u + sn / w * pu, (-w if kk > 0 else w) * sn * u + c * pu
        x, px = plane(x, px, k)
        y, py = plane(y, py, -k)
    else:
        x, y = x + s * px, y + s * py
    return [x, px, y, py, z + s * d / gamma ** 2, d]


def _moments(X):
    X = torch.stack(list(X)) if not torch.is_tensor(X) else X
    mean = X.mean(dim=1)
    c = X - mean[:, None]
    cov = c @ c.T / X.shape[1]
    iu = torch.triu_indices(6, 6)
    return torch.cat([mean, cov[iu[0], iu[1]]])


def _track(X, case, nodes, lattice, ks=None, diag=None, steps=None):
    """The split-operator steps on rows X (a list of six); ks: strengths as a tensor (thin)."""
    gamma = 1.0 + KIN_MEV / MASS_MEV
    C = QM_QEEV / ((gamma - 1.0) * (gamma + 1.0))
    q = math.copysign(CHARGE_C, QM_QEEV) / X[0].numel()
    slices = []
    for e, (kind, k, ds, ns) in enumerate(lattice):
        slices += [(kind, k, ds / ns, e)] * (ns if kind != THIN else 1)
    for t in range(case["steps"] if steps is None else steps):
        kind, k, L, e = slices[t % len(slices)]
        kq = k if ks is None else ks[e]
        X = _half(X, kind, k, L / 2, kq, gamma)
        pos = [X[0], X[2], X[4]]
        origin, h, hr = _geometry(pos, nodes, gamma)
        rho = _deposit(pos, origin, h, nodes, case["shape"], q)
        _, E = _field(rho, hr, nodes, case["op"] == "direct")
        Ep = _gather(pos, E, origin, h, nodes, case["shape"])
        X = [X[0], X[1] + C * L * Ep[0], X[2], X[3] + C * L * Ep[1], X[4],
             X[5] + gamma * C * L * Ep[2]]
        X = _half(X, kind, k, L / 2, None, gamma)
        if diag is not None:
            diag.append(_moments(X))
    return X


def _start(n, halo, seed):
    xi = _draws(n, halo, seed)
    return xi, [xi[a] * SIGMA[a] for a in range(6)]


def exact(case, seed):
    """The plain method in float64 torch: scattered deposits, torch's FFTs, the integrated
    Green's function's corner sums, autograd for the gradients."""
    nodes = (case["nx"], case["ny"], case["nz"])
    gamma = 1.0 + KIN_MEV / MASS_MEV
    if case["op"] == "batch":
        ns, gs, ks = _scan(case, seed)
        out = []
        for b, (nb, gb, kb) in enumerate(zip(ns, gs, ks)):
            _, X = _start(nb, 0.0, seed * 1000 + b)
            X = _track(X, case, (gb,) * 3, ((THIN, kb, 0.5, 1), (THIN, -kb, 0.5, 1)))
            out.append(torch.stack(X).reshape(-1))
        return torch.cat(out)
    xi, X = _start(case["n"], case["halo"], seed)
    lattice = _lattice(case)
    if case["op"] == "binned":
        del xi
        X = _track(X, case, nodes, lattice)
        pos = [X[0], X[2], X[4]]
        origin, h, _ = _geometry(pos, nodes, gamma)
        q = math.copysign(CHARGE_C, QM_QEEV) / case["n"]
        return {"rho": _deposit(pos, origin, h, nodes, case["shape"], q), "moments": _moments(X)}
    if case["op"] == "calls":
        X = _half(X, THIN, 0.0, 0.25, 1.0, gamma)
        pos = [X[0], X[2], X[4]]
        origin, h, hr = _geometry(pos, nodes, gamma)
        q = math.copysign(CHARGE_C, QM_QEEV) / case["n"]
        C = QM_QEEV / ((gamma - 1.0) * (gamma + 1.0))
        rho = _deposit(pos, origin, h, nodes, case["shape"], q)
        phi, E = _field(rho, hr, nodes, False)
        Ep = _gather(pos, E, origin, h, nodes, case["shape"])
        X = [X[0], X[1] + 0.5 * C * Ep[0], X[2], X[3] + 0.5 * C * Ep[1], X[4],
             X[5] + 0.5 * gamma * C * Ep[2]]
        X = _half(X, DRIFT, 0.0, 0.25, None, gamma)
        return {"rho": rho, "phi": phi, "E": E, "Ep": Ep, "X": torch.stack(X)}
    if case["op"] == "adjoint":
        if case["lattice"] != "quads8" or case["n"] * case["steps"] * (case["shape"] + 1) ** 3 > 6e8:
            return None
        X0 = torch.stack(X).requires_grad_()
        ks = torch.tensor([e[1] for e in lattice], dtype=torch.float64,
                          device="cuda").requires_grad_()
        X = torch.stack(_track(list(X0), case, nodes, lattice, ks=ks))
        c = X - X.mean(dim=1, keepdim=True)
        S = c @ c.T / X.shape[1]
        m = torch.stack([S[0, 0].sqrt(), S[2, 2].sqrt(),
                         (S[0, 0] * S[1, 1] - S[0, 1] ** 2).sqrt(),
                         (S[2, 2] * S[3, 3] - S[2, 3] ** 2).sqrt()])
        lam, dk = torch.autograd.grad(m.sum(), (X0, ks))
        return {"m": m.detach(), "dk": dk, "lam": lam, "dL": lam @ xi.T, "X": X.detach()}
    diag = [] if case["op"] == "diag" else None
    X = torch.stack(_track(X, case, nodes, lattice, diag=diag))
    if case["op"] == "diag":
        return {"diag": torch.stack(diag), "X": X}
    return {"X": X, "moments": _moments(X)}
