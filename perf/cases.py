"""The calls of this library that programs spend their time in, as cases that
can be timed and checked: short trajectories from a stored configuration, single
force evaluations, structure factors, the observables of a snapshot and a served
batch of small systems.

A case is a dict of plain values.  ``kind`` says which entry points a pass goes
through:

``traj``    ``rbsog_step`` for ``nsteps`` steps from a stored state (NVE or with
            a bath, with or without the energy history)
``forces``  ``rbsog_compute_forces`` with the near part and an energy row
``rho``     ``rbsog_compute_rho``: the structure factors of a step's modes
``ssf``     ``rbsog_ssf``: the static structure factor by lattice shell
``pairs``   a snapshot's other observables: pair histogram, displacements,
            mean squared displacement and velocity autocorrelation
``serve``   a served ensemble: admit ``nreq`` requests, step them to their end,
            retire them all

Reduced units as in ``workloads``: number density 3 / (4 pi), unit charges and
masses (a mixture has a tenth of its particles with q = 5, m = 20).
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2501_10946_amd as R

DEV = "cuda"

# Decompositions of Algorithm 1 at eps = 1e-4, by (kappa, r_c): h, t0, w, M1, M2.
SOG = {
    1.0: (3.0, 0.8981259380414027, 0.058648411400838735, 1.0154971619443622, 3, -1),
    0.5: (4.0, 0.922269402912814, 0.7448053913031851, 1.0176028668508228, 5, -2),
    0.1: (5.0, 0.9419093609279544, 0.8157742875708516, 1.0179975448750522, 8, -3),
}
BATHS = {"none": R.RBSOG_BATH_NONE, "langevin": R.RBSOG_BATH_LANGEVIN, "nose-hoover": R.RBSOG_BATH_NOSE_HOOVER}


def listed():
    return [
        # the smallest system of the suite with its energy record: a step is a
        # chain of short launches, so latency and launch count decide
        dict(name="traj 1e3", kind="traj", N=1000, kappa=1.0, gamma=1.0, P=100, mixed=False, mix=False, aspect=1.0,
             bath="none", energies=True, nsteps=20),
        # equilibration of a mid-size system: cuboid box, Langevin bath, mixed precision, odd sizes
        dict(name="traj 1e4 langevin cuboid", kind="traj", N=10007, kappa=0.5, gamma=10.0, P=193, mixed=True,
             mix=False, aspect=1.5, bath="langevin", energies=False, nsteps=20),
        # the N = 1e5 plasma, plain NVE production: lists live for several steps
        dict(name="traj 1e5", kind="traj", N=100000, kappa=0.5, gamma=10.0, P=200, mixed=False, mix=False, aspect=1.0,
             bath="none", energies=False, nsteps=20),
        # the binary mixture under a Nose-Hoover bath with its energy record
        dict(name="traj 2e5 mixture", kind="traj", N=200000, kappa=0.5, gamma=5.0, P=300, mixed=False, mix=True,
             aspect=1.0, bath="nose-hoover", energies=True, nsteps=10),
        # the headline plasma, hot: lists rebuilt at every step
        dict(name="traj 1e6", kind="traj", N=1000000, kappa=0.1, gamma=0.1, P=500, mixed=False, mix=False,
             aspect=1.0, bath="none", energies=False, nsteps=5),
        # the headline plasma, cold, in mixed precision with its energy record
        dict(name="traj 1e6 mixed", kind="traj", N=1000000, kappa=0.1, gamma=100.0, P=500, mixed=True, mix=False,
             aspect=1.0, bath="none", energies=True, nsteps=5),
        # one force evaluation of a small mixture for an outside integrator
        dict(name="forces 5e3", kind="forces", N=5003, kappa=0.5, gamma=5.0, P=300, mixed=False, mix=True,
             aspect=1.0),
        # one force evaluation of a large plasma
        dict(name="forces 3e5", kind="forces", N=300000, kappa=0.1, gamma=1.0, P=500, mixed=False, mix=False,
             aspect=1.0),
        # the structure factors of one step alone
        dict(name="rho 2.6e5", kind="rho", N=262147, kappa=0.1, gamma=1.0, P=500, mixed=False, mix=False, aspect=1.0),
        # the static structure factor of a snapshot over 4 000 lattice modes
        dict(name="ssf 2e4", kind="ssf", N=20000, kappa=0.5, gamma=10.0, m_s=100),
        # a snapshot's pair histogram, displacements and correlations
        dict(name="pairs 2e5", kind="pairs", N=200000, kappa=0.5, gamma=10.0, P=200, nbins=200),
        # sixteen requests of 500 to 5e4 particles served together, mixed precision as served
        dict(name="serve 16", kind="serve", nreq=16, sizes=104, nsteps=20, P=200, mixed=True),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["traj", "traj", "traj", "forces", "forces", "rho", "ssf", "pairs", "serve"])
    kappa = rng.choice([1.0, 0.5, 0.1])
    gamma = round(math.exp(rng.uniform(math.log(0.1), math.log(100.0))), 3)
    P = {1.0: 100, 0.5: 200, 0.1: 500}[kappa] if rng.random() < 0.4 else rng.randint(20, 500)
    if kind == "serve":
        return dict(kind=kind, nreq=rng.randint(3, 16), sizes=rng.randint(1, 999), nsteps=rng.randint(5, 20),
                    P=rng.randint(50, 200), mixed=rng.random() < 0.8)
    if kind == "ssf":
        return dict(kind=kind, N=log_int(500, 1e5), kappa=kappa, gamma=gamma, m_s=log_int(10, 100))
    if kind == "pairs":
        return dict(kind=kind, N=log_int(1000, 3e5), kappa=kappa, gamma=gamma, P=50, nbins=rng.randint(20, 1000))
    N = log_int(1000, 1e6 if kind == "rho" else 5e5)
    case = dict(kind=kind, N=N, kappa=kappa, gamma=gamma, P=P, mixed=rng.random() < 0.4, mix=rng.random() < 0.3,
                aspect=rng.choice([1.0, 1.0, 1.3]) if N > 3000 else 1.0)
    if kind == "traj":
        case |= dict(bath=rng.choice(["none", "none", "langevin", "nose-hoover"]), energies=rng.random() < 0.5,
                     nsteps=rng.randint(3, 20 if N < 2e5 else 6))
    return case


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def edges(case):
    """Box edges at the reduced density; ``aspect`` stretches z against x and y."""
    a = case.get("aspect", 1.0)
    Lx = (4.0 * math.pi * case["N"] / 3.0 / a) ** (1.0 / 3.0)
    return (Lx, Lx, Lx * a)


def generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def positions(N, L, gamma, g):
    """Weakly coupled: uniform.  Strongly coupled (gamma >= 1): the sites of a
    lattice with random displacements, so that no two particles overlap."""
    Lt = torch.tensor(L, dtype=torch.float64, device=DEV)[:, None]
    if gamma < 1.0:
        x = torch.rand((3, N), generator=g, dtype=torch.float64, device=DEV)
    else:
        side = (L[0] * L[1] * L[2] / N) ** (1.0 / 3.0)
        n = [math.ceil(e / side) for e in L]
        site = torch.randperm(n[0] * n[1] * n[2], generator=g, device=DEV)[:N]
        grid = torch.stack([site % n[0], site // n[0] % n[1], site // (n[0] * n[1])]).double()
        jitter = 0.15 * torch.randn((3, N), generator=g, dtype=torch.float64, device=DEV)
        x = torch.remainder((grid + 0.5 + jitter) / torch.tensor(n, dtype=torch.float64, device=DEV)[:, None], 1.0)
    x = x * Lt
    return torch.where(x >= Lt, torch.zeros_like(x), x).contiguous()


def particles(case, seed):
    """x, v [3, N] and q, m [N] of a case."""
    g = generator(seed)
    N = case["N"]
    x = positions(N, edges(case), case["gamma"], g)
    q = torch.ones(N, dtype=torch.float64, device=DEV)
    m = torch.ones(N, dtype=torch.float64, device=DEV)
    if case.get("mix"):
        q[N - N // 10:] = 5.0
        m[N - N // 10:] = 20.0
    v = torch.randn((3, N), generator=g, dtype=torch.float64, device=DEV) * torch.sqrt(1.0 / (case["gamma"] * m))
    v -= (v * m).sum(1, keepdim=True) / m.sum()
    return x, v.contiguous(), q, m


def decomposition(kappa):
    r_c, h, t0, w, M1, M2 = SOG[kappa]
    return R.sog_from_parameters(1.0 / kappa, r_c, h, t0, w, M1, M2)


def system(case, q, m, seed):
    L = edges(case)
    return R.System(q, m, L if case.get("aspect", 1.0) != 1.0 else L[0], decomposition(case["kappa"]),
                    1.0 / case["gamma"], case["P"], seed=seed,
                    precision=R.RBSOG_MIXED if case.get("mixed") else R.RBSOG_FP64)


DT = 0.01


def bath_of(case):
    return case.get("bath", "none")


def request_sizes(case):
    g = np.random.Generator(np.random.Philox(key=np.array([case["sizes"], 5], dtype=np.uint64)))
    return [int(round(math.exp(g.uniform(math.log(500), math.log(5e4))))) for _ in range(case["nreq"])]


def requests(case, seed):
    """The served requests: the case's sizes, log-uniform in [500, 5e4], couplings
    in [0.1, 100], screening uniform in [0.1, 2], host arrays as a server holds them."""
    g = np.random.Generator(np.random.Philox(key=np.array([seed, 3], dtype=np.uint64)))
    out = []
    for i, N in enumerate(request_sizes(case)):
        gamma = math.exp(g.uniform(math.log(0.1), math.log(100.0)))
        kappa = g.uniform(0.1, 2.0)
        L = (4.0 * math.pi * N / 3.0) ** (1.0 / 3.0)
        n = math.ceil(N ** (1.0 / 3.0))
        site = g.permutation(n ** 3)[:N]
        x = np.stack([site % n, site // n % n, site // (n * n)]) + 0.5 + 0.15 * g.standard_normal((3, N))
        x = np.ascontiguousarray(np.mod(x / n, 1.0) * L)
        x[x >= L] = 0.0
        sog = R.rbsog_sog_init(1.0 / kappa, 4.0, 1e-4)
        par = R.make_params(N, L, 1.0 / gamma, case["P"], seed, replica=i,
                            precision=R.RBSOG_MIXED if case["mixed"] else R.RBSOG_FP64)
        v = np.ascontiguousarray(g.standard_normal((3, N)) / math.sqrt(gamma))
        out.append((par, sog, x, v, np.ones(N), np.ones(N)))
    return out


def prepare(case, seed):
    if case["kind"] == "serve":
        reqs = requests(case, seed)
        need = sum(R.rbsog_ens_bytes(p, s, case["nsteps"]) for p, s, *_ in reqs)
        total = sum(r[2].shape[1] for r in reqs)
        return dict(case=case, reqs=reqs, ens=Ensemble(need, case["nreq"]),
                    x=np.empty((total * 3,)), v=np.empty((total * 3,)),
                    e=np.empty((case["nreq"], case["nsteps"], R.ENERGY_COLS)))
    x, v, q, m = particles(case, seed)
    s = dict(case=case, x=x, q=q)
    if case["kind"] == "ssf":
        s["scratch"] = torch.empty(R.rbsog_ssf_scratch_size(case["N"], case["m_s"]) // 8 + 32, dtype=torch.float64,
                                   device=DEV)
        s["s"] = torch.empty(case["m_s"] + 1, dtype=torch.float64, device=DEV)
        return s
    sys_ = s["sys"] = system(case, q, m, seed)
    if case["kind"] == "rho":
        s["rho"] = torch.empty((case["P"], 2), dtype=torch.float64, device=DEV)
    elif case["kind"] == "pairs":
        s["hist"] = torch.empty(case["nbins"], dtype=torch.int64, device=DEV)
        s["disp"] = torch.zeros_like(x)
        s["x_last"] = torch.remainder(x - 0.1 * v, edges(case)[0]).contiguous()
        s["v"] = v
        s["v0"] = v.flip(1).contiguous()
        s["scratch"] = torch.empty(R.rbsog_msd_scratch_size() // 8, dtype=torch.float64, device=DEV)
        s["out"] = torch.empty(2, dtype=torch.float64, device=DEV)
    else:
        s["f"] = torch.empty_like(x)
        s["e"] = torch.zeros(R.ENERGY_COLS, dtype=torch.float64, device=DEV)
        if case["kind"] == "forces":
            s["f_near"] = torch.empty_like(x)
        else:   # the stored configuration a trajectory starts from, with its force
            R.rbsog_compute_forces(sys_.h, 0, x, s["f"], None, None)
            s |= dict(x0=x.clone(), v0=v, f0=s["f"].clone(), v=v.clone())
            if case["energies"]:
                s["eh"] = torch.empty((case["nsteps"], R.ENERGY_COLS), dtype=torch.float64, device=DEV)
    return s


class Ensemble:
    """The server's ensemble, kept from batch to batch."""

    def __init__(self, pool_bytes, slots):
        self.slots = slots
        self.h = R.rbsog_ens_create(pool_bytes + (1 << 20), slots)

    def __del__(self):
        if R is not None and getattr(self, "h", None):
            R.rbsog_ens_destroy(self.h)


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def run(s):
    case = s["case"]
    return {"traj": run_traj, "forces": run_forces, "rho": run_rho, "ssf": run_ssf, "pairs": run_pairs,
            "serve": run_serve}[case["kind"]](case, s)


def run_traj(case, s):
    h = s["sys"].h
    s["x"].copy_(s["x0"])
    s["v"].copy_(s["v0"])
    s["f"].copy_(s["f0"])
    if bath_of(case) != "none":   # selecting a bath starts its state afresh
        R.rbsog_set_bath(h, BATHS[bath_of(case)], 1.0, 1.0 / case["gamma"])
    R.rbsog_step(h, s["x"], s["v"], s["f"], 0, case["nsteps"], DT, s.get("eh"))
    out = dict(x=s["x"], v=s["v"], f=s["f"])
    if case["energies"]:
        out["energy"] = s["eh"]
    return out


def run_forces(case, s):
    R.rbsog_compute_forces(s["sys"].h, 0, s["x"], s["f"], s["f_near"], s["e"])
    return dict(f=s["f"], f_near=s["f_near"], energy=s["e"])


def run_rho(case, s):
    R.rbsog_compute_rho(s["sys"].h, 0, s["x"], s["rho"])
    return s["rho"]


def run_ssf(case, s):
    R.rbsog_ssf(s["x"], s["q"], edges(case)[0], case["m_s"], s["scratch"], s["s"])
    return s["s"]


def run_pairs(case, s):
    L = edges(case)[0]
    s["hist"].zero_()
    R.rbsog_rdf(s["sys"].h, s["x"], SOG[case["kappa"]][0], case["nbins"], s["hist"])
    R.rbsog_track(s["x"], L, s["x_last"], s["disp"])
    R.rbsog_msd_vacf(s["disp"], s["v0"], s["v"], s["scratch"], s["out"])
    return dict(hist=s["hist"], disp=s["disp"], msd_vacf=s["out"])


def run_serve(case, s):
    ens = s["ens"]
    slot_of = {}
    for i, (par, sog, x, v, q, m) in enumerate(s["reqs"]):
        slot_of[R.rbsog_ens_admit(ens.h, par, sog, x, v, q, m, case["nsteps"], 0.005)] = i
    for _ in range(case["nsteps"]):
        R.rbsog_ens_step(ens.h)
    offset = np.cumsum([0] + [3 * r[2].shape[1] for r in s["reqs"]])
    while slot_of:
        for slot in R.rbsog_ens_poll(ens.h, ens.slots):
            i = slot_of.pop(slot)
            a, b = offset[i], offset[i + 1]
            R.rbsog_ens_retire(ens.h, slot, s["x"][a:b], s["v"][a:b], s["e"][i])
    return dict(x=s["x"], v=s["v"], energy=s["e"])


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

PAIR_FLOPS = 60.0        # difference, r^2, 1/r, the pair function, three accumulations
PHASE_FLOPS = 30.0       # phase, reduction, sine or cosine pair, accumulation


def work(case):
    kind = case["kind"]
    if kind == "serve":
        n = sum(request_sizes(case))   # r_c = 4: 63 neighbours
        it = n * case["nsteps"]
        return dict(bytes=n * 8 * (8 + 6), flops=it * (63 * PAIR_FLOPS + 2 * case["P"] * PHASE_FLOPS))
    N = case["N"]
    if kind == "ssf":
        modes = 4.0 / 3.0 * math.pi * case["m_s"] ** 1.5
        return dict(bytes=8.0 * 4 * N, flops=N * modes * PHASE_FLOPS)
    near = SOG[case["kappa"]][0] ** 3 - 1.0 / N   # neighbours within r_c at density 3 / (4 pi)
    if kind == "rho":
        return dict(bytes=8.0 * 4 * N, flops=N * case["P"] * PHASE_FLOPS)
    if kind == "pairs":
        return dict(bytes=8.0 * N * (3 + 3 + 6 + 6 + 6), flops=N * near * 15.0)
    per = near * PAIR_FLOPS + 2.0 * case["P"] * PHASE_FLOPS
    if kind == "forces":
        return dict(bytes=8.0 * N * (3 + 1 + 6), flops=N * per)
    return dict(bytes=8.0 * N * (9 * 2 + 9 + 2), flops=case["nsteps"] * N * per)


# ---------------------------------------------------------------------------
# the same results in 64 bits, from the formulas alone
# ---------------------------------------------------------------------------

def exact(case, seed):
    kind = case["kind"]
    if kind == "serve":
        return None
    x, v, q, m = particles(case, seed)
    L = edges(case)
    if kind == "ssf":
        n = lattice_cube(case["m_s"])[1]
        rho = structure_factors(x, q, L, n)
        mm = torch.from_numpy((n.astype(np.int64) ** 2).sum(1)).to(DEV)
        s = torch.zeros(case["m_s"] + 1, dtype=torch.float64, device=DEV)
        c = torch.zeros_like(s)
        s.index_add_(0, mm, (rho.abs() ** 2))
        c.index_add_(0, mm, torch.ones_like(mm, dtype=torch.float64))
        return s / c.clamp(min=1.0)
    if kind == "pairs":
        last = torch.remainder(x - 0.1 * v, L[0])
        d = x - last
        d = d - L[0] * torch.round(d / L[0])
        return dict(hist=None, disp=d, msd_vacf=torch.stack([(d * d).sum(), (v.flip(1) * v).sum()]) / case["N"])
    if kind == "traj" and case["N"] * case["nsteps"] > 2.2e6:
        return None
    E = Reference(case, q, seed)
    if kind == "rho":
        n, _ = E.modes(0)
        rho = structure_factors(x, q, L, n)
        return torch.stack([rho.real, rho.imag], 1)
    if kind == "forces":
        f, fn, e = E.force(x, 0)
        return dict(f=f, f_near=fn, energy=torch.tensor(e, dtype=torch.float64, device=DEV))
    dt, kT, bath = DT, 1.0 / case["gamma"], bath_of(case)
    Lt = torch.tensor(L, dtype=torch.float64, device=DEV)[:, None]
    f = E.force(x, 0)[0]
    xi, eta, gkT, rows = 0.0, 0.0, 3.0 * case["N"] * kT, []

    def half(v, xi):   # Nose-Hoover half-step, unit relaxation time
        K = 0.5 * float((m * v * v).sum())
        xi += 0.25 * dt * (2.0 * K - gkT) / gkT
        sc = math.exp(-0.5 * dt * xi)
        xi += 0.25 * dt * (2.0 * K * sc * sc - gkT) / gkT
        return v * sc, xi

    for n in range(case["nsteps"]):
        if bath == "nose-hoover":
            v, xi = half(v, xi)
        v = v + 0.5 * dt / m * f
        if bath == "langevin":
            c1 = math.exp(-dt)
            x = x + 0.5 * dt * v
            v = c1 * v + torch.sqrt((1.0 - c1 * c1) * kT / m) * normals(case["N"], n + 1, seed)
            x = x + 0.5 * dt * v
        else:
            x = x + dt * v
        x = torch.remainder(x, Lt)
        f, _, e = E.force(x, n + 1)
        v = v + 0.5 * dt / m * f
        if bath == "nose-hoover":
            v, xi = half(v, xi)
        e[5] = 0.5 * float((m * v * v).sum())
        rows.append(e)
    out = dict(x=x, v=v, f=f)
    if case["energies"]:
        out["energy"] = torch.tensor(rows, dtype=torch.float64, device=DEV)
    return out


def philox(c0, c1, c2, seed):
    """Philox4x64-10 at counters (c0, c1, c2, 0), key (seed, 0): four words each."""
    def mul(a, b):   # high and low words of a 64 x 64 product
        a0, a1 = a & np.uint64(0xFFFFFFFF), a >> np.uint64(32)
        b0, b1 = np.uint64(b & 0xFFFFFFFF), np.uint64(b >> 32)
        t = a0 * b0
        u = a1 * b0 + (t >> np.uint64(32))
        w = a0 * b1 + (u & np.uint64(0xFFFFFFFF))
        return a1 * b1 + (u >> np.uint64(32)) + (w >> np.uint64(32)), a * np.uint64(b)

    c0 = np.asarray(c0, dtype=np.uint64)
    c = [c0, np.full_like(c0, c1), np.full_like(c0, c2), np.zeros_like(c0)]
    k0, k1, mask = seed, 0, (1 << 64) - 1
    for _ in range(10):
        hA, lA = mul(c[0], 0xD2E7470EE14C6C93)
        hB, lB = mul(c[2], 0xCA5A826395121157)
        c = [hB ^ c[1] ^ np.uint64(k0), lB, hA ^ c[3] ^ np.uint64(k1), lA]
        k0, k1 = (k0 + 0x9E3779B97F4A7C15) & mask, (k1 + 0xBB67AE8584CAA73B) & mask
    return c


def normals(N, step, seed):
    u = [((w >> np.uint64(11)).astype(np.float64) + 1.0) * 2.0 ** -53 for w in philox(np.arange(N), step, 1, seed)]
    r0, r1 = np.sqrt(-2.0 * np.log(u[0])), np.sqrt(-2.0 * np.log(u[2]))
    t = 2.0 * math.pi
    return torch.from_numpy(np.stack([r0 * np.cos(t * u[1]), r0 * np.sin(t * u[1]), r1 * np.cos(t * u[3])])).to(DEV)


def lattice_cube(mmax):
    """Shell sizes r3(0..mmax) and the points 1 <= |n|^2 <= mmax by (|n|^2, nx, ny, nz)."""
    r = int(math.isqrt(mmax))
    a = np.arange(-r, r + 1, dtype=np.int32)
    m = (a[:, None, None] ** 2 + a[None, :, None] ** 2 + a[None, None, :] ** 2).ravel()
    keep = np.flatnonzero((m >= 1) & (m <= mmax))
    order = keep[np.argsort(m[keep], kind="stable")]
    w = 2 * r + 1
    n = np.stack([order // (w * w) - r, order // w % w - r, order % w - r], 1)
    return np.bincount(m[keep], minlength=mmax + 1), n


def structure_factors(x, q, L, n):
    """sum_j q_j exp(i k.r_j) of the integer modes n [P, 3] (complex [P])."""
    s = x / torch.tensor(L, dtype=torch.float64, device=DEV)[:, None]
    nt = torch.from_numpy(np.ascontiguousarray(n)).double().to(DEV)
    rho = torch.zeros(len(n), dtype=torch.complex128, device=DEV)
    step = max(1, (1 << 25) // x.shape[1])
    for a in range(0, len(n), step):
        u = nt[a:a + step] @ s
        u = 2.0 * math.pi * (u - torch.round(u))
        rho[a:a + step] = torch.complex((q * torch.cos(u)).sum(1), (q * torch.sin(u)).sum(1))
    return rho


class Reference:
    """Forces and energies of one system from the method's formulas (near pairs
    within r_c, the random batch's modes), FP64 torch operations."""

    def __init__(self, case, q, seed):
        self.case, self.q, self.seed = case, q, seed
        self.L = edges(case)
        self.V = self.L[0] * self.L[1] * self.L[2]
        r_c, h, t0, w, M1, M2 = SOG[case["kappa"]]
        self.r_c, self.lam = r_c, 1.0 / case["kappa"]
        self.c, self.s, self.A, self.B = [], [], [], []
        for j in range(-M1, M2 + 1):
            t = t0 + j * h
            c = h / math.sqrt(math.pi) * math.exp(0.5 * t - math.exp(-t) / (4.0 * self.lam ** 2)) * (w if j == M2 else 1.0)
            s = math.exp(t)
            self.c.append(c)
            self.s.append(s)
            self.A.append(math.pi * math.sqrt(math.pi) * c / (s * math.sqrt(s)))
            self.B.append(1.0 / (4.0 * s))
        self.Q1, self.Q2 = float(q.sum()), float((q * q).sum())
        self.table()

    def fhat(self, k2):
        return sum(a * np.exp(-b * k2) for a, b in zip(self.A, self.B))

    def table(self):
        """The sampling measure: entries (points or shells) in order with their
        weights; entry i of a cube holds the points of one shell."""
        L, thr = self.L, 1e-16 * self.fhat(0.0)
        if L[0] == L[2]:
            t = 2.0 * math.pi / L[0]
            tk2 = t * t
            m = np.arange(1, 512 * 512, dtype=np.float64)
            mmax = int(np.flatnonzero(self.fhat(tk2 * m) < thr)[0])
            size, self.pts = lattice_cube(mmax)
            shell = np.flatnonzero(size)
            self.count, k2 = size[shell], tk2 * shell
            self.first = np.cumsum(self.count) - self.count
        else:
            k2max = 1.0
            while self.fhat(k2max) >= thr:
                k2max *= 1.1
            r = [int(e * math.sqrt(k2max) / (2.0 * math.pi)) + 1 for e in L]
            a = np.stack(np.meshgrid(*[np.arange(-i, i + 1) for i in r], indexing="ij"), -1).reshape(-1, 3)
            k = [2.0 * math.pi * a[:, d] / L[d] for d in range(3)]
            k2 = k[0] * k[0] + k[1] * k[1] + k[2] * k[2]
            keep = np.flatnonzero((self.fhat(k2) >= thr) & (k2 > 0.0))
            keep = keep[np.lexsort((a[keep, 2], a[keep, 1], a[keep, 0], k2[keep]))]
            self.pts, k2 = a[keep], k2[keep]
            self.count, self.first = np.ones(len(keep), dtype=np.int64), np.arange(len(keep))
        kTV = self.V / self.case["gamma"]
        F = kTV / (kTV / self.Q2 + self.lam ** 2 / (1.0 + self.lam ** 2 * k2))
        self.cdf = np.cumsum(self.count * F * self.fhat(k2))
        self.coef = self.cdf[-1] / ((self.case["P"] * self.V) * F)

    def modes(self, step):
        w = philox(np.arange(self.case["P"]), step, 0, self.seed)
        target = (w[0] >> np.uint64(11)).astype(np.float64) * 2.0 ** -53 * self.cdf[-1]
        i = np.minimum(np.searchsorted(self.cdf, target, side="right"), len(self.cdf) - 1)
        j = np.array([(int(a) * int(b)) >> 64 for a, b in zip(w[1], self.count[i])])
        return self.pts[self.first[i] + j], self.coef[i]

    def pair(self, d, qq):
        """Force factor and energy of pairs at displacement d [3, ...] (0 beyond r_c)."""
        r2 = (d * d).sum(0)
        ok = (r2 < self.r_c ** 2) & (r2 > 0.0)
        r2 = torch.where(ok, r2, torch.ones_like(r2))
        r = torch.sqrt(r2)
        y = torch.exp(-r / self.lam)
        fac, en = y * (1.0 + r / self.lam) / (r2 * r), y / r
        for c, s in zip(self.c, self.s):
            g = torch.exp(-s * r2)
            fac = fac - 2.0 * c * s * g
            en = en - c * g
        w = torch.where(ok, qq, torch.zeros_like(qq))
        return fac * w, en * w, r2

    def near(self, x):
        """Near forces, energy and virial by cells of at least r_c, padded to the fullest."""
        N, L, q = x.shape[1], self.L, self.q
        nc = [int(e / self.r_c) for e in L]
        Lt = torch.tensor(L, dtype=torch.float64, device=DEV)
        nt = torch.tensor(nc, device=DEV)
        c = torch.minimum((x / Lt[:, None] * nt[:, None]).long(), nt[:, None] - 1)
        cid = (c[2] * nc[1] + c[1]) * nc[0] + c[0]
        order = torch.argsort(cid, stable=True)
        count = torch.bincount(cid, minlength=nc[0] * nc[1] * nc[2])
        cap, start = int(count.max()), torch.cumsum(count, 0) - count
        member = torch.full((len(count), cap), -1, device=DEV)
        slot = torch.arange(N, device=DEV) - start[cid[order]]
        member[cid[order], slot] = order
        f, en, vir = torch.zeros_like(x), 0.0, 0.0
        cells = torch.arange(len(count), device=DEV)
        cz, cy, cx = cells // (nc[0] * nc[1]), cells // nc[0] % nc[1], cells % nc[0]
        step = max(1, (1 << 24) // (cap * cap))
        offsets = {((a % nc[0]), (b % nc[1]), (e % nc[2])) for a in (-1, 0, 1) for b in (-1, 0, 1) for e in (-1, 0, 1)}
        for a, b, e in sorted(offsets):
            other = ((cz + e) % nc[2] * nc[1] + (cy + b) % nc[1]) * nc[0] + (cx + a) % nc[0]
            for lo in range(0, len(count), step):
                i, j = member[lo:lo + step], member[other[lo:lo + step]]
                live = (i[:, :, None] >= 0) & (j[:, None, :] >= 0)
                d = x[:, i][:, :, :, None] - x[:, j][:, :, None, :]
                d = d - Lt[:, None, None, None] * torch.round(d / Lt[:, None, None, None])
                fac, u, r2 = self.pair(d, torch.where(live, q[i][:, :, None] * q[j][:, None, :], 0.0))
                g = (fac * d).sum(-1)
                f.index_add_(1, i.clamp(min=0).reshape(-1), torch.where(i >= 0, g, 0.0).reshape(3, -1))
                en += 0.5 * float(u.sum())
                vir += 0.5 * float((fac * r2).sum())
        return f, en, vir

    def far(self, x, step):
        n, coef = self.modes(step)
        L = torch.tensor(self.L, dtype=torch.float64, device=DEV)
        rho = structure_factors(x, self.q, self.L, n)
        nt, cf = torch.from_numpy(np.ascontiguousarray(n)).double().to(DEV), torch.from_numpy(coef).to(DEV)
        k = 2.0 * math.pi * nt / L
        s = x / L[:, None]
        f = torch.zeros_like(x)
        chunk = max(1, (1 << 25) // x.shape[1])
        for a in range(0, len(nt), chunk):
            u = nt[a:a + chunk] @ s
            u = 2.0 * math.pi * (u - torch.round(u))
            r = rho[a:a + chunk]
            im = cf[a:a + chunk, None] * (r.imag[:, None] * torch.cos(u) - r.real[:, None] * torch.sin(u))
            f -= k[a:a + chunk].T @ im
        k2 = (k * k).sum(1)
        ex = [torch.exp(-b * k2) for b in self.B]
        F = sum(a * e for a, e in zip(self.A, ex))
        G = sum(a * b * e for a, b, e in zip(self.A, self.B, ex))
        u = cf * rho.abs() ** 2
        return f * self.q, 0.5 * float(u.sum()), float((u * (1.5 - k2 * G / F)).sum())

    def force(self, x, step):
        fn, un, wn = self.near(x)
        ff, uf, wf = self.far(x, step)
        row = [un, uf, sum(self.A) * self.Q1 ** 2 / (2.0 * self.V), -0.5 * sum(self.c) * self.Q2,
               -(self.Q1 ** 2) * 4.0 * math.pi * self.lam ** 2 / (2.0 * self.V), 0.0, wn, wf]
        return fn + ff, fn, row
