"""The work a user of the photon-transport library has it do, as timed cases.

Every case goes through the public binding (`paper_2302_12727_amd.rt.RT` and
`rollout`), on seeded synthetic inputs made on the device.  A case's fields:

  kind       "step"     one RT step: injection, gradient, transport and the
                        photon totals (the path a simulation spends its time in)
             "rebuild"  a start or a moved particle set: rt_build_cells and
                        rt_set_sources at new positions, then one step
             "ticks"    one full cycle of individual time steps (rt_tick)
             "adjoint"  one rt_adjoint call, its records given
             "rollout"  differentiable rollout, forward and backward, with
                        checkpoints
             "operators" photon removal and drift correction of one step
  points     "lattice" (n_side^3 jittered lattice, as the Iliev-type tests) or
             "clustered" (Plummer profile plus 10% background, glass-like)
  size       particles per side (lattice) or nominal number (clustered)
  groups, precision ("fp64" or "fp32c"), sources, solver ("glf", "hll"),
  surfaces ("hopkins", "ivanova")

`exact` evaluates the same equations (arXiv:2302.12727, Parts II and III) in
64 bits with plain torch on neighbour pairs found by brute force.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2302_12727_amd.rollout import RolloutBuffers, rollout
from paper_2302_12727_amd.rt import ETA, KAPPA, RT

CFL, C_RED = 0.9, 1.0
PLUMMER_SCALE, PLUMMER_CUT, BACKGROUND = 0.05, 0.5, 0.1
#: Neighbours r < max(H_k, H_l) and gather neighbours r < H_i of one particle, on average.
NEIGHBOURS, GATHER = 46.8, 39.0
#: The most particles whose pairs `exact` finds by brute force.
EXACT_MAX = 240_000


def _case(name, kind, points, size, groups, precision="fp64", sources=0, solver="glf",
          surfaces="hopkins", steps=1):
    return dict(name=name, kind=kind, points=points, size=size, groups=groups, precision=precision,
                sources=sources, solver=solver, surfaces=surfaces, steps=steps)


def listed():
    return [
        # the smallest run of the tests: launches and latency set its time
        _case("step_lattice16_g1", "step", "lattice", 16, 1),
        # the Iliev-suite resolution with the three ionising groups: the headline
        _case("step_lattice128_g3", "step", "lattice", 128, 3, sources=16),
        # the same in compensated FP32
        _case("step_lattice128_g3_fp32c", "step", "lattice", 128, 3, "fp32c", sources=16),
        # an odd size (no full last block) with the other Riemann solver
        _case("step_lattice61_g2_hll", "step", "lattice", 61, 2, sources=3, solver="hll"),
        # a clustered FP64 run around one central source
        _case("step_clustered_g3", "step", "clustered", 1_000_000, 3, sources=1),
        # the clustered four-group run of the large adjoint workload, forward
        _case("step_clustered_g4_fp32c", "step", "clustered", 150_000, 4, "fp32c", sources=256),
        # and one backward step of it
        _case("adjoint_clustered_g4_fp32c", "adjoint", "clustered", 60_000, 4, "fp32c", sources=64),
        # source inversion: 20 steps with a checkpoint every 5, forward and backward
        _case("rollout_lattice64_g3", "rollout", "lattice", 64, 3, sources=64, steps=20),
        # individual power-of-two time steps where the resolution varies
        _case("ticks_clustered_g3", "ticks", "clustered", 100_000, 3, sources=1),
        # starting the headline run, or moving its particles
        _case("rebuild_lattice128_g3", "rebuild", "lattice", 128, 3, sources=16),
        # moving a small clustered set, where the build's latency counts
        _case("rebuild_clustered_g1_fp32c", "rebuild", "clustered", 20_000, 1, "fp32c", sources=1),
        # the two per-particle operators beside the transport
        _case("operators_lattice128_g3", "operators", "lattice", 128, 3),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "step", "rebuild", "ticks", "adjoint", "rollout",
                       "operators"])
    points = rng.choice(["lattice", "clustered"])
    groups = rng.choice([1, 2, 3, 3, 4, 5])
    precision = "fp64" if kind == "rollout" else rng.choice(["fp64", "fp32c"])
    top = {"rollout": 60, "ticks": 60, "adjoint": 100}.get(kind, 110)
    if kind == "adjoint" and precision == "fp32c":
        top = 40
    side = _log_uniform(rng, 12, top)
    size = side if points == "lattice" else _log_uniform(rng, max(2000, side ** 3 // 2), side ** 3 + 2001)
    solver = rng.choice(["glf", "glf", "hll"])
    surfaces = rng.choice(["hopkins", "hopkins", "ivanova"])
    c = _case("", kind, points, size, groups, precision, rng.choice([1, 3, 16, 64]), solver,
              surfaces, rng.choice([3, 7, 10]) if kind == "rollout" else 1)
    del c["name"]
    return c


# ---------------------------------------------------------------------------
# inputs

def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _gen(seed, what):
    return torch.Generator(device=_device()).manual_seed(1_000_003 * what + int(seed))


@functools.lru_cache(maxsize=16)
def _leaf_cells(nominal):
    """(lower corners, sides) of the cells that hold one particle each: the
    unit box split in octants while a cell would hold over 4 particles at the
    largest density of the Plummer profile plus background in its sphere."""
    a, rc = PLUMMER_SCALE, PLUMMER_CUT
    m_max = rc ** 3 / (rc * rc + a * a) ** 1.5
    side = 1.0
    lo = np.zeros((1, 3))
    out_lo, out_side = [], []
    octants = np.array([[i, j, k] for i in (0, 1) for j in (0, 1) for k in (0, 1)], dtype=float)
    while lo.size:
        r = np.maximum(np.sqrt(((lo + 0.5 * side - 0.5) ** 2).sum(axis=1)) - 0.5 * side, 0.0)
        rho = BACKGROUND + np.where(r < rc, (1 - BACKGROUND) * 3 / (4 * math.pi * a ** 3 * m_max)
                                    * (1 + (r / a) ** 2) ** -2.5, 0.0)
        split = (nominal * rho * side ** 3 > 4.0) | (side > 0.13)
        out_lo.append(lo[~split])
        out_side.append(np.full((~split).sum(), side))
        side *= 0.5
        lo = (lo[split][:, None, :] + side * octants[None]).reshape(-1, 3)
    return np.concatenate(out_lo), np.concatenate(out_side)


def _count(case):
    return case["size"] ** 3 if case["points"] == "lattice" else len(_leaf_cells(case["size"])[1])


def _positions(case, seed):
    dev, g = _device(), _gen(seed, 1)
    if case["points"] == "lattice":
        k = case["size"]
        ax = torch.arange(k, dtype=torch.float64, device=dev)
        x = torch.stack(torch.meshgrid(ax, ax, ax, indexing="ij"), dim=-1).reshape(-1, 3)
        x = x + 0.5 + 0.2 * (torch.rand(x.shape, generator=g, dtype=torch.float64, device=dev) - 0.5)
        x = x / k
    else:
        lo, side = (torch.from_numpy(v).to(dev) for v in _leaf_cells(case["size"]))
        u = torch.rand(lo.shape, generator=g, dtype=torch.float64, device=dev)
        x = lo + (0.5 + 0.5 * (u - 0.5)) * side[:, None]
        x = x + torch.rand((1, 3), generator=g, dtype=torch.float64, device=dev)
        # no spatial order in the input, as in a snapshot
        x = x[torch.randperm(x.shape[0], generator=g, device=dev)]
    x = torch.remainder(x, 1.0)
    return torch.where(x >= 1.0, torch.zeros_like(x), x).contiguous()


def _fields(case, seed, what=2, fmax=0.9, negative=0.0):
    """Radiation states [n, G, 4]: E log-normal, F isotropic with |F| up to
    fmax c E; the given share of the energies with the sign changed."""
    dev, g = _device(), _gen(seed, what)
    n, G = _count(case), case["groups"]
    rnd = lambda *s: torch.rand(*s, generator=g, dtype=torch.float64, device=dev)
    nrm = lambda *s: torch.randn(*s, generator=g, dtype=torch.float64, device=dev)
    E = torch.exp(nrm(n, G))
    d = nrm(n, G, 3)
    F = (fmax * C_RED * E * rnd(n, G) / d.norm(dim=-1))[..., None] * d
    if negative > 0:
        E = torch.where(rnd(n, G) < negative, -1e-3 * E, E)
    U = torch.cat([E[..., None], F], dim=-1)
    return U.to(_dtype(case))


def _dtype(case):
    return torch.float64 if case["precision"] == "fp64" else torch.float32


def _sources(case, seed, x):
    """Source positions on particles, luminosities log-uniform on [0.01, 1]."""
    S, dev, g = case["sources"], _device(), _gen(seed, 4)
    if not S:
        return None, None
    pick = torch.randperm(x.shape[0], generator=g, device=dev)[:S]
    L = torch.rand((S, case["groups"]), generator=g, dtype=torch.float64, device=dev)
    return x[pick].contiguous(), torch.exp(math.log(1e-2) * L)


def _cotangent(case, seed):
    g = _gen(seed, 5)
    lam = torch.randn((_count(case), case["groups"], 4), generator=g, dtype=torch.float64,
                      device=_device())
    return lam.to(_dtype(case))


def _absorbers(case, seed):
    """Densities of three species at both ends of the step, the group cross
    sections (optical depths of about 1e-3 per step) and the displacements."""
    dev, g = _device(), _gen(seed, 6)
    n, G = _count(case), case["groups"]
    rnd = lambda *s: torch.rand(*s, generator=g, dtype=torch.float64, device=dev)
    n_old, n_new, sigma = rnd(n, 3), rnd(n, 3), rnd(G, 3) * 1e-3 * n ** (1 / 3)
    return n_old, n_new, sigma, (rnd(n, 3) - 0.5) * 0.2 * n ** (-1 / 3)


# ---------------------------------------------------------------------------
# the measured calls

def prepare(case, seed):
    x = _positions(case, seed)
    rt = RT(x.shape[0], case["groups"], case["precision"], c_red=C_RED, cfl=CFL)
    xs, L = _sources(case, seed, x)
    s = {"case": case, "rt": rt, "x": x, "xs": xs, "L": L, "U": _fields(case, seed),
         "Ub": rt.state(), "UD": rt.grad_buffer(),
         "Q": torch.zeros(case["groups"], dtype=torch.float64, device=x.device)}
    rt.rt_set_riemann(case["solver"])
    kind = case["kind"]
    if kind == "rebuild":
        return s
    rt.rt_build_cells(x)
    rt.rt_set_surfaces(case["surfaces"])
    rt.rt_set_sources(xs)
    if kind == "ticks":
        _, s["cycle"] = rt.rt_time_bins(8)
        rt.rt_gradient(s["U"], s["UD"])
        s["acc"] = torch.zeros(s["U"].shape, dtype=torch.float64, device=x.device)
    elif kind == "adjoint":
        rt.rt_gradient(s["U"], s["UD"])
        s["Uu"] = _fields(case, seed, 3, 1.02, 1e-3)      # the forward's unguarded update
        s["lam"] = _cotangent(case, seed)
    elif kind == "rollout":
        s["bufs"] = RolloutBuffers(rt, case["steps"], 5)
        s["lam"] = _cotangent(case, seed)
    elif kind == "operators":
        s["n_old"], s["n_new"], s["sigma"], s["dx"] = _absorbers(case, seed)
        rt.rt_gradient(s["U"], s["UD"])
        s["absorbed"] = torch.zeros_like(s["Q"])
        s["Qd"] = torch.zeros_like(s["Q"])
    return s


def run(s):
    rt, kind = s["rt"], s["case"]["kind"]
    if kind == "step":
        rt.step(s["U"], s["L"], UD=s["UD"], U_out=s["Ub"], photon_total=s["Q"])
        return {"U": s["Ub"], "Q": s["Q"]}
    if kind == "rebuild":
        perm, h, V, dt = rt.rt_build_cells(s["x"])
        if not s.get("surfaces"):                        # kept by later builds
            s["surfaces"] = s["case"]["surfaces"]
            rt.rt_set_surfaces(s["surfaces"])
        rt.rt_set_sources(s["xs"])
        rt.step(s["U"], s["L"], UD=s["UD"], U_out=s["Ub"], photon_total=s["Q"])
        return {"perm": perm, "h": h, "V": V, "dt": dt, "U": s["Ub"], "Q": s["Q"]}
    if kind == "ticks":
        for t in range(s["cycle"]):
            rt.rt_tick(s["U"], s["L"], t, s["UD"], s["acc"], photon_total=s["Q"])
        return {"U": s["U"], "Q": s["Q"]}
    if kind == "adjoint":
        dL = torch.zeros_like(s["L"])
        lam = rt.rt_adjoint(None, s["L"], s["lam"], UD=s["UD"], U_unguarded=s["Uu"], dL_dL=dL)
        return {"lam": lam, "dL": dL}
    if kind == "rollout":
        L = s["L"].clone().requires_grad_(True)
        U0 = s["U"].detach().requires_grad_(True)
        U = rollout(rt, L, U0, s["case"]["steps"], 5, s["bufs"])
        gL, gU = torch.autograd.grad(U, (L, U0), s["lam"])
        return {"U": U.detach(), "dL": gL, "dU": gU}
    rt.rt_absorb(s["U"], s["n_old"], s["sigma"], n_new=s["n_new"], photon_total=s["Q"],
                 absorbed=s["absorbed"])
    rt.rt_drift(s["UD"], s["dx"], s["Ub"], photon_total=s["Qd"])
    return {"U": s["U"], "Q": s["Q"], "moved": s["Ub"], "Qd": s["Qd"]}


def work(case):
    """Bytes and operations of one pass: states, gradient records and geometry
    records once per operator that reads or writes them; 74 + 179 G operations
    per pair of the transport, 26 + 28 G per gather neighbour of the gradient,
    about 2.5 times the transport per pair of its adjoint."""
    n, G, kind = _count(case), case["groups"], case["kind"]
    w = 8 if case["precision"] == "fp64" else 4
    state, record, geometry = 4 * G * w, 16 * G * w, 96
    pairs = 0.5 * NEIGHBOURS
    step_b = n * (2 * state + record + geometry)
    step_f = n * (pairs * (74 + 179 * G) + GATHER * (26 + 28 * G))
    back_b = n * (3 * state + record + geometry)
    back_f = n * (pairs * 2.5 * (74 + 179 * G) + GATHER * (26 + 28 * G))
    if kind == "step":
        return {"bytes": step_b, "flops": step_f}
    if kind == "rebuild":
        return {"bytes": step_b + n * (24 + 8 + 8 + 8 + geometry),
                "flops": step_f + n * GATHER * 60}
    if kind == "ticks":
        # a particle takes one step of its own per 2^bin ticks
        own = 1.0
        if case["points"] == "clustered":
            side = _leaf_cells(case["size"])[1]
            own = float((side.max() / side).mean())
        return {"bytes": own * step_b, "flops": own * step_f}
    if kind == "adjoint":
        return {"bytes": back_b, "flops": back_f}
    if kind == "rollout":
        k = case["steps"]
        again = k - (1 + (k - 1) % 5)                    # recomputed by the backward
        return {"bytes": (k + again) * step_b + k * back_b, "flops": (k + again) * step_f + k * back_f}
    return {"bytes": n * (2 * state + 48 + 8) + n * (record + state + 24 + 8),
            "flops": n * G * (4 + 12 + 24)}


# ---------------------------------------------------------------------------
# the same in 64 bits with plain torch

def _w(q):
    return torch.clamp(1 - q, min=0) ** 3 - 4 * torch.clamp(0.5 - q, min=0) ** 3


def _dw(q):
    return -3 * torch.clamp(1 - q, min=0) ** 2 + 12 * torch.clamp(0.5 - q, min=0) ** 2


def _image(s):
    return s - torch.round(s)


def _nearest(points, x, k):
    """Distances and indices of the k nearest x of each point."""
    k = min(k, x.shape[0])
    rows = max(1, 200_000_000 // x.shape[0])
    dist, idx = [], []
    for p in points.split(rows):
        r2 = torch.zeros((p.shape[0], x.shape[0]), dtype=x.dtype, device=x.device)
        for a in range(3):
            r2 += _image(x[None, :, a] - p[:, None, a]) ** 2
        d, i = torch.topk(r2, k, dim=1, largest=False)
        dist.append(d.sqrt())
        idx.append(i)
    return torch.cat(dist), torch.cat(idx)


def _smoothing(dist):
    """Roots h of h^3 sum_j W(r_j, kappa h) = eta^3 for rows of distances."""
    def g(h):
        H = KAPPA * h
        return (16 / math.pi / KAPPA ** 3) * _w(dist / H[:, None]).sum(1) - ETA ** 3

    lo = torch.zeros_like(dist[:, 0])
    hi = dist[:, -1] / KAPPA
    for _ in range(80):
        mid = 0.5 * (lo + hi)
        up = g(mid) < 0
        lo, hi = torch.where(up, mid, lo), torch.where(up, hi, mid)
    return 0.5 * (lo + hi)


def _morton(x):
    key = torch.zeros(x.shape[0], dtype=torch.int64, device=x.device)
    q = (x * 2097152.0).to(torch.int64).clamp(0, 2097151)
    for b in range(21):
        for a in range(3):
            key |= ((q[:, a] >> b) & 1) << (3 * b + 2 - a)
    return torch.argsort(key, stable=True)


class _Geometry:
    """Static geometry in Morton order: smoothing lengths, volumes, matrices,
    gather entries (i, j) and directed pairs (k, l) with their surfaces."""

    def __init__(self, case, seed):
        x0 = _positions(case, seed)
        self.perm = _morton(x0)
        x = self.x = x0[self.perm]
        n = self.n = x.shape[0]
        dist, idx = _nearest(x, x, 160)
        self.h = _smoothing(dist)
        H = self.H = KAPPA * self.h
        near = (dist < H[:, None]) & (idx != torch.arange(n, device=x.device)[:, None])
        self.gi, col = torch.nonzero(near, as_tuple=True)
        self.gj = idx[self.gi, col]
        s = _image(x[self.gj] - x[self.gi])
        r = s.norm(dim=1)
        w = _w(r / H[self.gi])
        norm = 16 / math.pi / H ** 3
        add = lambda v: torch.zeros((n,) + v.shape[1:], dtype=x.dtype, device=x.device).index_add(0, self.gi, v)
        self.V = 1 / (norm * (0.5 + add(w)))
        psi = w * (norm * self.V)[self.gi]
        B = torch.linalg.inv(add(psi[:, None, None] * s[:, :, None] * s[:, None, :]))
        self.tilde = (B[self.gi] @ s[:, :, None])[..., 0] * psi[:, None]
        self.dt = CFL * torch.min((3 * self.V / (4 * math.pi)) ** (1 / 3)) / C_RED
        # directed pairs: the gather entries and their mirrors, once each
        key = torch.unique(torch.cat([self.gi * n + self.gj, self.gj * n + self.gi]))
        k, l = self.k, self.l = key // n, key % n
        s = self.s = _image(x[l] - x[k])
        r = s.norm(dim=1)
        if case["surfaces"] == "ivanova":
            sg = _image(x[self.gj] - x[self.gi])
            rg = sg.norm(dim=1)
            g = add(-((norm / H)[self.gi] * _dw(rg / H[self.gi]) / rg)[:, None] * sg)

            def grad_psi(i, s):
                q = r / H[i]
                gw = -(norm / H)[i, None] * _dw(q)[:, None] * (s / r[:, None])
                return self.V[i, None] * gw - (self.V[i] ** 2 * norm[i] * _w(q))[:, None] * g[i]
            A = self.V[k, None] * grad_psi(k, s) - self.V[l, None] * grad_psi(l, -s)
        else:
            def tilde(i, s):
                return (B[i] @ s[:, :, None])[..., 0] * (_w(r / H[i]) * norm[i] * self.V[i])[:, None]
            A = self.V[k, None] * tilde(k, s) - self.V[l, None] * tilde(l, -s)
        self.A, self.An = A, A.norm(dim=1)
        self.wk = (self.h[k] / (self.h[k] + self.h[l]))[:, None]

    def sources(self, case, seed):
        """(gas, source, xi / V) of the injection."""
        xs, L = _sources(case, seed, self.x[torch.argsort(self.perm)])
        if xs is None:
            return None, None
        dist, idx = _nearest(xs, self.x, 160)
        H = KAPPA * _smoothing(dist)
        src, col = torch.nonzero(dist < H[:, None], as_tuple=True)
        gas = idx[src, col]
        w = _w(dist[src, col] / H[src])
        s = _image(self.x[gas] - xs[src])
        octant = ((s >= 0) * torch.tensor([1, 2, 4], device=s.device)).sum(1)
        wa = torch.zeros((len(xs), 8), dtype=w.dtype, device=w.device).index_put(
            (src, octant), w, accumulate=True)
        xi = w / ((wa > 0).sum(1)[src] * wa[src, octant])
        return (gas, src, xi / self.V[gas]), L


def _guard(q):
    E = torch.clamp(q[..., 0], min=0)
    F = q[..., 1:]
    F2 = (F * F).sum(-1)
    over = F2 > (C_RED * E) ** 2
    F = F * torch.where(over, C_RED * E / torch.sqrt(torch.where(over, F2, torch.ones_like(F2))),
                        torch.ones_like(E))[..., None]
    return torch.cat([E[..., None], torch.where((E == 0)[..., None], torch.zeros_like(F), F)], -1)


def _flux(q, A):
    """(F.A, c^2 P A) of the M1 closure."""
    E, F = q[..., 0], q[..., 1:]
    f = F / torch.where(E > 0, C_RED * E, torch.ones_like(E))[..., None]
    f2 = (f * f).sum(-1)
    d = 1 / (2 + torch.sqrt(torch.clamp(4 - 3 * f2, min=0)))
    FA = (F * A).sum(-1)
    a = C_RED ** 2 * E * (1 / 3 - f2 * d)
    b = 3 * C_RED * d * (f * A).sum(-1)
    return torch.cat([FA[..., None], a[..., None] * A + b[..., None] * F], -1)


@functools.lru_cache(maxsize=1)
def _speed_table():
    """Extreme eigenvalues of the M1 flux Jacobian along n, 65 x 65 nodes in
    (|F|/cE, cos(F, n)), by complex-step differentiation."""
    f, mu = np.meshgrid(np.linspace(0, 1, 65), np.linspace(-1, 1, 65), indexing="ij")
    U = np.zeros(f.shape + (4,))
    U[..., 0], U[..., 1], U[..., 2] = 1.0, f * mu, f * np.sqrt(1 - mu * mu)
    J = np.zeros(f.shape + (4, 4))
    for m in range(4):
        q = U.astype(complex)
        q[..., m] += 1e-30j
        E, F = q[..., 0], q[..., 1:]
        F2 = (F * F).sum(-1)
        D = 2 * E + np.sqrt(4 * E * E - 3 * F2)
        J[..., 0, m] = F[..., 0].imag / 1e-30
        for a in range(3):
            J[..., 1 + a, m] = ((E / 3 - F2 / D) * (a == 0) + 3 * F[..., 0] / D * F[..., a]).imag / 1e-30
    ev = np.linalg.eigvals(J).real
    tab = np.stack([ev.min(-1), ev.max(-1)], -1)
    tab[0] = [-1 / math.sqrt(3), 1 / math.sqrt(3)]
    tab[-1] = mu[-1][:, None]
    return tab


def _speeds(q, A, An):
    tab = torch.from_numpy(_speed_table()).to(q.device)
    E, F = q[..., 0], q[..., 1:]
    F2 = (F * F).sum(-1)
    ok = (E > 0) & (F2 > 0)
    one, zero = torch.ones_like(E), torch.zeros_like(E)
    Fn = torch.sqrt(torch.where(ok, F2, one))
    f = torch.where(ok, torch.clamp(Fn / (C_RED * torch.where(ok, E, one)), max=1), zero)
    mu = torch.where(ok, torch.clamp((F * A).sum(-1) / (Fn * An), -1, 1), zero)
    u, v = f * 64, (mu + 1) * 32
    i, j = (t.detach().floor().long().clamp(0, 63) for t in (u, v))
    tu, tv = (u - i)[..., None], (v - j)[..., None]
    lam = (1 - tu) * ((1 - tv) * tab[i, j] + tv * tab[i, j + 1]) \
        + tu * ((1 - tv) * tab[i + 1, j] + tv * tab[i + 1, j + 1])
    return C_RED * lam[..., 0], C_RED * lam[..., 1]


def _gradient(geo, U):
    d = (U[geo.gj] - U[geo.gi])[..., None] * geo.tilde[:, None, :]
    return torch.zeros(U.shape + (3,), dtype=U.dtype, device=U.device).index_add(0, geo.gi, d)


def _sum_flux(geo, U, D, solver, weight=None):
    """sum_l Flux_kl . A_kl of one group (U [n, 4], D [n, 4, 3]), each pair
    times `weight` if given."""
    k, l = geo.k, geo.l
    a = (D[k] * geo.s[:, None, :]).sum(-1)
    b = (D[l] * geo.s[:, None, :]).sum(-1)
    m = torch.where(a * b > 0, torch.where(a.abs() <= b.abs(), a, b), torch.zeros_like(a))
    qL, qR = _guard(U[k] + geo.wk * m), _guard(U[l] - (1 - geo.wk) * m)
    fL, fR = _flux(qL, geo.A), _flux(qR, geo.A)
    if solver == "glf":
        P = 0.5 * (fL + fR) - 0.5 * C_RED * geo.An[:, None] * (qR - qL)
    else:
        (lo1, hi1), (lo2, hi2) = _speeds(qL, geo.A, geo.An), _speeds(qR, geo.A, geo.An)
        lp = torch.clamp(torch.maximum(hi1, hi2), min=0)
        lm = torch.clamp(torch.minimum(lo1, lo2), max=0)
        ok = lp > lm
        den = torch.where(ok, lp - lm, torch.ones_like(lp))
        half = torch.full_like(lp, 0.5)
        w1, w2 = torch.where(ok, lp / den, half), torch.where(ok, -lm / den, half)
        w3 = torch.where(ok, lp * lm * geo.An / den, torch.zeros_like(lp))
        P = w1[:, None] * fL + w2[:, None] * fR + w3[:, None] * (qR - qL)
    if weight is not None:
        P = P * weight[:, None]
    return torch.zeros_like(U).index_add(0, k, P)


def _inject(geo, src, U, L, dt):
    """U [n, G, 4] after the injection over dt (a number, or one per particle)."""
    if src is None:
        return U
    gas, s, coef = src
    dt = dt[gas] if torch.is_tensor(dt) and dt.dim() else dt
    add = torch.zeros(U.shape[:2], dtype=U.dtype, device=U.device).index_add(
        0, gas, (coef * dt)[:, None] * L[s])
    return torch.cat([(U[..., 0] + add)[..., None], U[..., 1:]], -1)


def _unguarded(geo, U, solver):
    out = []
    for g in range(U.shape[1]):
        u = U[:, g]
        out.append(u - (geo.dt / geo.V)[:, None] * _sum_flux(geo, u, _gradient(geo, u), solver))
    return torch.stack(out, 1)


def _total(geo, U):
    return (geo.V[:, None] * U[..., 0]).sum(0)


def _cycle(geo, case, src, L, U):
    """One full cycle of individual time steps, bins at most 8 and at most 2
    apart between neighbours."""
    n = geo.n
    tau = CFL * (3 * geo.V / (4 * math.pi)) ** (1 / 3) / C_RED
    b = torch.zeros(n, dtype=torch.int64, device=U.device)
    for e in range(1, 9):
        b += (geo.dt * 2.0 ** e <= tau) & (b == e - 1)
    while True:
        low = b.scatter_reduce(0, geo.k, b[geo.l] + 2, "amin")
        if torch.equal(low, b):
            break
        b = low
    pair = torch.minimum(b[geo.k], b[geo.l])
    D = torch.stack([_gradient(geo, U[:, g]) for g in range(U.shape[1])], 1)
    acc = torch.zeros_like(U)
    Us = U.clone()                                       # the states the neighbours see
    own, both = geo.dt * torch.exp2(b.double()), geo.dt * torch.exp2(pair.double())
    for t in range(1 << int(b.max())):
        ends = (t + 1) % (1 << b) == 0
        U = torch.where(ends[:, None, None], _inject(geo, src, Us, L, own), Us)
        due = ((t + 1) % (1 << pair) == 0) * both
        for g in range(U.shape[1]):
            D[:, g] = torch.where(ends[:, None, None], _gradient(geo, U[:, g]), D[:, g])
            acc[:, g] += _sum_flux(geo, U[:, g], D[:, g], case["solver"], due)
        new = _guard(U - acc / geo.V[:, None, None])
        Us = torch.where(ends[:, None, None], new, U)
        acc = torch.where(ends[:, None, None], torch.zeros_like(acc), acc)
    return Us


def exact(case, seed):
    n = _count(case)
    if case["kind"] == "operators":
        return _exact_operators(case, seed) if n <= EXACT_MAX else None
    heavy = {"ticks": 130_000, "rollout": 30_000, "adjoint": 130_000}.get(case["kind"], EXACT_MAX)
    if n > heavy:
        return None
    geo = _Geometry(case, seed)
    src, L = geo.sources(case, seed)
    U0 = _fields(case, seed).double()
    if case["kind"] in ("step", "rebuild"):
        U = _guard(_unguarded(geo, _inject(geo, src, U0, L, geo.dt), case["solver"]))
        out = {"U": U, "Q": _total(geo, U)}
        if case["kind"] == "rebuild":
            out.update(perm=None, h=geo.h, V=geo.V, dt=geo.dt.reshape(1))
        return out
    if case["kind"] == "ticks":
        U = _cycle(geo, case, src, L, U0)
        return {"U": U, "Q": _total(geo, U)}
    lam = _cotangent(case, seed).double()
    Lv = L.clone().requires_grad_(True)
    if case["kind"] == "adjoint":
        # the guard's derivative at the given unguarded states; the records
        # hold the state after the injection
        Uu = _fields(case, seed, 3, 1.02, 1e-3).double().requires_grad_(True)
        (lg,) = torch.autograd.grad(_guard(Uu), Uu, lam)
        gU = []
        for g in range(case["groups"]):
            U1 = U0[:, g].clone().requires_grad_(True)
            u = U1[:, None, :]
            (d,) = torch.autograd.grad(_unguarded(geo, u, case["solver"])[:, 0], U1, lg[:, g])
            gU.append(d)
        gU = torch.stack(gU, 1)
        (gL,) = torch.autograd.grad(_inject(geo, src, U0, Lv, geo.dt), Lv, gU)
        return {"lam": gU, "dL": gL}
    states = [U0]
    with torch.no_grad():
        for _ in range(case["steps"]):
            U = _inject(geo, src, states[-1], L, geo.dt)
            states.append(_guard(_unguarded(geo, U, case["solver"])))
    gL = torch.zeros_like(L)
    for U in reversed(states[:-1]):
        with torch.no_grad():
            U1 = _inject(geo, src, U, L, geo.dt)
        back = []
        for g in range(case["groups"]):
            u = U1[:, g].clone().requires_grad_(True)
            nxt = _guard(_unguarded(geo, u[:, None, :], case["solver"]))[:, 0]
            back.append(torch.autograd.grad(nxt, u, lam[:, g])[0])
        lam = torch.stack(back, 1)
        gL += torch.autograd.grad(_inject(geo, src, U, Lv, geo.dt), Lv, lam)[0]
    return {"U": states[-1], "dL": gL, "dU": lam}


def _exact_operators(case, seed):
    geo = _Geometry(case, seed)
    U = _fields(case, seed).double()
    D = torch.stack([_gradient(geo, U[:, g]) for g in range(U.shape[1])], 1)
    n_old, n_new, sigma, dx = _absorbers(case, seed)
    depth = C_RED * geo.dt * 0.5 * (n_old + n_new) @ sigma.T
    left = U * torch.clamp(1 - depth, min=0)[..., None]
    moved = _guard(U + (D * dx[:, None, None, :]).sum(-1))
    return {"U": left, "Q": _total(geo, left), "moved": moved, "Qd": _total(geo, moved)}
