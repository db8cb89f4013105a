"""Timed cases of the framework: what a program that uses it has it do, over the
range of lattices, precisions and entry points.

``listed()`` gives the fixed cases, ``draw(rng)`` one more of the same ranges,
``prepare`` the handle a program keeps (a random start made from the seed),
``run`` one pass through the public entry points, ``work`` what a pass cannot do
without, and ``exact`` the same chain in plain 64-bit torch.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2106_11286_amd import mcheis as M


# ---------------------------------------------------------------------------
# Cases.  Fields: do (chain / exchange / block / snapshot); kind, Lx, Ly, Lz,
# mask (periodic axes), R (sphere radius in cells, 0: whole box); sizes (edge
# lengths that the replicas of an uneven batch take in turn, "" otherwise);
# prec; reps; J, K, axis, T and T1 (temperatures evenly spaced over the
# replicas); n, m (chain: unmeasured and measured sweeps; exchange: rounds and
# sweeps per round; block: block size and steps); api (chain: "schedule", or
# "sweep" with the last record read back).
# ---------------------------------------------------------------------------
def _case(name, do, kind, L, mask=7, R=0.0, sizes="", prec="f32", reps=1, K=0.02, axis="z",
          T=1.4, T1=None, n=0, m=1, api="sweep"):
    return {"name": name, "do": do, "kind": kind, "Lx": L[0], "Ly": L[1], "Lz": L[2],
            "mask": mask, "R": float(R), "sizes": sizes, "prec": prec, "reps": reps, "J": 1.0,
            "K": K, "axis": axis, "T": T, "T1": T if T1 is None else T1, "n": n, "m": m,
            "api": api}


def listed():
    return [
        # a small lattice followed sweep by sweep in FP64 (validation runs,
        # trajectories): every sweep's record comes back
        _case("sc16-f64-trajectory", "chain", "sc", (16, 16, 16), prec="f64", K=0.1, T=1.2, n=0,
              m=64, api="schedule"),
        # the smallest calls: one measured sweep of a film-like lattice with
        # open faces and odd edges, its record read back, as a program that
        # watches or steers a run does
        _case("sc-film-one-sweep", "chain", "sc", (50, 37, 23), mask=0, K=0.1, T=0.9, n=0, m=1),
        # a temperature ladder of small replicas in one handle, thermalised and
        # measured (finite-size scaling, Binder cumulants)
        _case("sc24-ladder-17", "chain", "sc", (24, 24, 24), reps=17, K=0.05, T=0.4, T1=2.0, n=32,
              m=32, api="schedule"),
        # many replicas of uneven size at their own temperatures, every sweep
        # measured: the batch that serves a whole study
        _case("sc-batch-64-uneven", "chain", "sc", (0, 0, 0), sizes="64 32 96 48 48 96 32 64",
              reps=64, K=0.1, T=0.8, T1=2.0, n=0, m=8),
        # replica exchange across the critical region
        _case("sc64-exchange-32", "exchange", "sc", (64, 64, 64), reps=32, K=0.01, T=1.41,
              T1=1.48, n=3, m=4),
        # the paper's own block scheme on its Fig. 1 lattice, with the count of
        # concurrent neighbours, for comparison with the colour sweep
        _case("sc128-block-scheme", "block", "sc", (128, 128, 128), K=0.01, T=1.3, n=8, m=16),
        # one temperature of the M(T) ladder: thermalisation and measurement
        _case("sc256-schedule", "chain", "sc", (256, 256, 256), K=0.05, T=1.2, n=8, m=8,
              api="schedule"),
        # 10^8 spins, every sweep measured, in both precisions
        _case("sc464-f32", "chain", "sc", (464, 464, 464), K=0.02, T=1.4, n=0, m=4),
        _case("sc464-f64", "chain", "sc", (464, 464, 464), prec="f64", K=0.02, T=1.4, n=0, m=2),
        # the other lattices: bcc at 10^8 spins, and an fcc nanoparticle with
        # an open surface (a 3.6 million-spin sphere in its box)
        _case("bcc368-f32", "chain", "bcc", (368, 368, 368), K=0.02, T=1.9, n=0, m=3),
        _case("fcc-particle-R60", "chain", "fcc", (128, 128, 128), mask=0, R=60.0, K=0.05,
              axis="111", T=0.9, n=4, m=4, api="schedule"),
        # analysis and checkpoint of a stored state: observables from scratch,
        # spins to natural order and back, on a film with odd edges
        _case("sc-film-snapshot", "snapshot", "sc", (302, 251, 211), mask=1, K=0.05, T=1.2),
    ]


MOST_UPDATES = 2.0e8  # updates of a drawn pass: at most what the largest listed FP64 case does


def _edges(rng, n_cells, even_x, periodic_even, mask):
    """Three edges of about n_cells cells, not all alike, odd ones where allowed."""
    c = n_cells ** (1.0 / 3.0)
    L = [max(4, int(round(c * math.exp(rng.uniform(-0.35, 0.35))))) for _ in range(3)]
    for a in range(3):
        if (a == 0 and even_x) or (periodic_even and (mask >> a) & 1):
            L[a] += L[a] % 2
    return tuple(L)


def draw(rng):
    do = rng.choice(["chain", "chain", "chain", "chain", "chain", "batch", "exchange", "block",
                     "snapshot"])
    prec = rng.choice(["f32", "f32", "f64"])
    K = round(rng.uniform(0.0, 0.1), 3)
    T = round(rng.uniform(0.6, 2.0), 3)
    if do in ("chain", "snapshot"):
        kind = rng.choice(["sc", "sc", "sc", "bcc", "fcc"])
        nb = {"sc": 1, "bcc": 2, "fcc": 4}[kind]
        sites = math.exp(rng.uniform(math.log(2.0e3), math.log(9.0e7 if prec == "f32" else 4.0e7)))
        mask = rng.choice([7, 7, 7, 3, 1, 0])
        L = _edges(rng, sites / nb, kind == "sc", kind == "sc", mask)
        R = 0.0
        if rng.random() < 0.2:  # a nanoparticle
            mask, R = 0, round(0.47 * min(L), 2)
        axis = "111" if kind == "fcc" else "z"
        N = L[0] * L[1] * L[2] * nb
        if do == "snapshot":
            return _drawn(_case("", "snapshot", kind, L, mask, R, prec=prec, K=K, axis=axis, T=T))
        total = max(1, min(48, int(MOST_UPDATES / N)))
        api = rng.choice(["schedule", "sweep"])
        n = rng.randint(0, total - 1) if total > 1 else 0
        return _drawn(_case("", "chain", kind, L, mask, R, prec=prec, K=K, axis=axis, T=T,
                            n=n, m=max(1, total - n), api=api))
    if do == "batch":
        reps = rng.choice([2, 3, 5, 8, 12, 16, 24, 32, 48])
        c = math.exp(rng.uniform(math.log(8), math.log(96)))
        sizes = sorted({max(6, 2 * int(round(0.5 * c * f))) for f in (0.5, 0.75, 1.0)})
        total = max(2, min(48, int(MOST_UPDATES / (reps * max(sizes) ** 3))))
        n = rng.randint(0, total - 1)
        return _drawn(_case("", "chain", "sc", (0, 0, 0), 7, sizes=" ".join(map(str, sizes)),
                            prec=prec, reps=reps, K=K, T=0.6, T1=2.0, n=n, m=total - n,
                            api=rng.choice(["schedule", "sweep"])))
    if do == "exchange":
        L = 2 * rng.randint(4, 36)
        return _drawn(_case("", "exchange", "sc", (L, L, L), prec=prec, reps=rng.randint(4, 32),
                            K=K, T=1.38, T1=1.5, n=rng.randint(1, 4), m=rng.randint(1, 6)))
    L = _edges(rng, math.exp(rng.uniform(math.log(3.0e4), math.log(1.0e7))), True, True, 7)
    return _drawn(_case("", "block", "sc", L, prec=prec, K=K, T=T, n=rng.choice([5, 8, 16]),
                        m=rng.randint(4, 24)))


def _drawn(c):
    del c["name"]
    return c


AXES = {"z": (0.0, 0.0, 1.0), "111": (1.0, 1.0, 1.0)}


def _replicas(case):
    reps = []
    sizes = [int(v) for v in case["sizes"].split()]
    T = np.linspace(case["T"], case["T1"], case["reps"])
    for r in range(case["reps"]):
        L = (sizes[r % len(sizes)],) * 3 if sizes else (case["Lx"], case["Ly"], case["Lz"])
        reps.append(dict(kind=case["kind"], L=L, periodic_mask=case["mask"],
                         sphere_radius=case["R"], J=case["J"], K=case["K"],
                         e=AXES[case["axis"]], T=float(T[r]), replica_id=r))
    return reps


def prepare(case, seed):
    sim = M.Simulation([M.Replica(**r) for r in _replicas(case)], precision=case["prec"],
                       seed=seed, init="random")
    if case["do"] == "exchange":
        sim.exchange_init()
    return {"case": case, "sim": sim, "step": 0}


def _spins(sim):
    """The current spins in the library's layout: the state's own planes, or,
    for a batch, one tensor per component."""
    planes = [sim.state_spins(r) for r in range(sim.n_reps)]
    if sim.n_reps == 1:
        return list(planes[0])
    with torch.cuda.stream(sim.stream):
        return [torch.cat([p[a] for p in planes]) for a in range(3)]


def _obs(obs):
    return [[o["M"], o["absM"], o["E"], o["E_exch"], o["E_anis"], o["n_accepted"]] for o in obs]


def run(state):
    case, sim = state["case"], state["sim"]
    if case["do"] == "chain":
        if case["api"] == "schedule":
            T = np.array([[r.T for r in sim.replicas]])
            rec = sim.run_schedule(T, n_equil=case["n"], n_meas=case["m"])
            return {"records": rec, "spins": _spins(sim)}
        if case["n"]:
            sim.sweep(case["n"])
        sim.sweep(case["m"], measure=True)
        obs = sim.observables()
        # one array for all replicas: M, |M|, E, E_exch, E_anis, accepted moves
        return {"observables": np.array([[*o[0], *o[1:]] for o in _obs(obs)], dtype=np.float64),
                "spins": _spins(sim)}
    if case["do"] == "exchange":
        sim.exchange_sweep(case["n"], case["m"])
        st = sim.exchange_state()
        return {"slots": np.array(st["replica_at_slot"]), "accepted": np.array(st["accepted"]),
                "spins": _spins(sim)}
    if case["do"] == "block":
        sim.block_steps(case["n"], state["step"], case["m"], conflicts=True, reset=True)
        state["step"] += case["m"]
        return {"counts": np.array(sim.block_counts()), "spins": _spins(sim)}
    obs = sim.measure_state()
    nat = sim.to_natural(0)
    sim.from_natural(0, nat)
    return {"observables": np.array([[*o[0], *o[1:5]] for o in _obs(obs)], dtype=np.float64),
            "natural": nat, "spins": _spins(sim)}


def _sites(r):
    nb = {"sc": 1, "bcc": 2, "fcc": 4}[r["kind"]]
    box = r["L"][0] * r["L"][1] * r["L"][2] * nb
    if r["sphere_radius"] > 0:
        return box, 4.0 / 3.0 * math.pi * r["sphere_radius"] ** 3 * nb
    return box, box


def work(case):
    """Bytes: a sweep reads and writes each spin once, also where a cache or
    the LDS can hold the state between sweeps of one call.  Operations of one
    attempted move: ten Philox rounds (two products, four exclusive ors), the
    proposal, the field of the neighbours, the energy difference, the
    acceptance test and the renormalisation."""
    esz = 4 if case["prec"] == "f32" else 8
    N = sum(_sites(r)[1] for r in _replicas(case))
    z = {"sc": 6, "bcc": 8, "fcc": 12}[case["kind"]]
    ops = 60 + 10 + 3 * z + 25 + 5 + 10
    if case["do"] == "snapshot":
        # state read for the observables; read and written by each conversion
        return {"bytes": 5.0 * 3 * esz * N, "flops": (3 * z + 10.0) * N}
    if case["do"] == "block":
        moves = float(N) / case["n"] * case["m"]
        return {"bytes": moves * 3 * esz * (z + 2), "flops": moves * ops}
    sweeps = case["n"] * case["m"] if case["do"] == "exchange" else case["n"] + case["m"]
    return {"bytes": 2.0 * 3 * esz * N * sweeps, "flops": float(ops) * N * sweeps}


# ---------------------------------------------------------------------------
# The same passes in plain 64-bit torch.
# ---------------------------------------------------------------------------
MASK32 = 0xFFFFFFFF


def _philox(c0, c1, c2, c3, seed):
    """Philox4x32-10 (Salmon et al., SC'11) on int64 tensors of 32-bit words."""
    k0, k1 = seed & MASK32, (seed >> 32) & MASK32
    for _ in range(10):
        pa, pb = c0 * 0xD2511F53, c2 * 0xCD9E8D57
        c0, c1, c2, c3 = (((pb >> 32) & MASK32) ^ c1 ^ k0, pb & MASK32,
                          ((pa >> 32) & MASK32) ^ c3 ^ k1, pa & MASK32)
        k0, k1 = (k0 + 0x9E3779B9) & MASK32, (k1 + 0xBB67AE85) & MASK32
    return c0, c1, c2, c3


def _words(s, rid, t, tag, seed):
    full = torch.full_like
    return _philox(s, full(s, rid), full(s, t), full(s, tag), seed)


def _u(w):
    return ((w >> 9).double() + 0.5) * 2.0 ** -23


def _sphere(w0, w1):
    z = 2.0 * _u(w0) - 1.0
    r = torch.sqrt(1.0 - z * z)
    phi = 2.0 * math.pi * _u(w1)
    return torch.stack([r * torch.cos(phi), r * torch.sin(phi), z])


BASIS = {"sc": [(0, 0, 0)], "bcc": [(0, 0, 0), (1, 1, 1)],
         "fcc": [(0, 0, 0), (1, 1, 0), (1, 0, 1), (0, 1, 1)]}


class _Exact:
    """One replica: S[b] of shape (3, Lz, Ly, Lx) for each basis site b."""

    def __init__(self, r, seed, dev):
        self.r, self.seed = r, seed
        self.Lx, self.Ly, self.Lz = r["L"]
        self.basis = BASIS[r["kind"]]
        self.sc = r["kind"] == "sc"
        nb = len(self.basis)
        shape = (self.Lz, self.Ly, self.Lx)
        cell = torch.arange(self.Lx * self.Ly * self.Lz, device=dev).view(shape)
        self.s = [cell * nb + b for b in range(nb)]
        ax = [torch.arange(n, device=dev) for n in (self.Lz, self.Ly, self.Lx)]
        self.parity = ((ax[0][:, None, None] + ax[1][:, None] + ax[2]) & 1) if self.sc else None
        self.occ = []
        for bx, by, bz in self.basis:
            if r["sphere_radius"] > 0:
                q2 = ((2 * ax[0] + bz - self.Lz)[:, None, None] ** 2 +
                      (2 * ax[1] + by - self.Ly)[:, None] ** 2 + (2 * ax[2] + bx - self.Lx) ** 2)
                self.occ.append(q2.double() <= 4.0 * r["sphere_radius"] ** 2)
            else:
                self.occ.append(torch.ones(shape, dtype=torch.bool, device=dev))
        e = np.array(r["e"], dtype=np.float64)
        self.e = [float(v) for v in e / np.linalg.norm(e)]
        self.T, self.t = r["T"], 0
        self.S = []
        for b in range(nb):
            w = _words(self.s[b], r["replica_id"], 0, 1, seed)
            self.S.append(_sphere(w[0], w[1]) * self.occ[b])
        self.N = int(sum(int(o.sum()) for o in self.occ))

    def _shift(self, A, o):
        """A at cell + o (z, y, x offsets in o), zero across open faces."""
        mask = self.r["periodic_mask"]
        for axis, (d, L, bit) in enumerate(zip(o, (self.Lz, self.Ly, self.Lx), (4, 2, 1))):
            if d == 0:
                continue
            A = torch.roll(A, -d, dims=1 + axis)
            if not mask & bit:
                at = [slice(None)] * 4
                at[1 + axis] = slice(L - d, L) if d > 0 else slice(0, -d)
                A[tuple(at)] = 0.0
        return A

    def bonds(self, b):
        """(b2, (dz, dy, dx)) of every neighbour of a site of basis b."""
        if self.sc:
            return [(0, o) for o in ((-1, 0, 0), (1, 0, 0), (0, -1, 0), (0, 1, 0), (0, 0, -1),
                                     (0, 0, 1))]
        out = []
        for b2, p2 in enumerate(self.basis):
            if b2 == b:
                continue
            d = [p2[a] - self.basis[b][a] for a in (2, 1, 0)]
            choice = [(0,) if v == 0 else (0, -v) for v in d]
            out += [(b2, (i, j, k)) for i in choice[0] for j in choice[1] for k in choice[2]]
        return out

    def field(self, b):
        h = torch.zeros_like(self.S[b])
        for b2, o in self.bonds(b):
            h += self._shift(self.S[b2], o)
        return h

    def attempt(self, S, h, w):
        """Proposal and decision from the words w: (new spins, accepted)."""
        new = _sphere(w[0], w[1])
        P = _u(w[2])
        e = self.e
        pn = new[0] * e[0] + new[1] * e[1] + new[2] * e[2]
        po = S[0] * e[0] + S[1] * e[1] + S[2] * e[2]
        dH = -self.r["J"] * (h * (new - S)).sum(0) - self.r["K"] * (pn * pn - po * po)
        acc = dH <= 0
        if self.T > 0:
            acc |= P <= torch.exp(-dH / self.T)
        return new / torch.sqrt((new * new).sum(0)), acc

    def sweep(self):
        n_acc = 0
        for c in range(2 if self.sc else len(self.basis)):
            b = 0 if self.sc else c
            w = _words(self.s[b], self.r["replica_id"], self.t, 0, self.seed)
            new, acc = self.attempt(self.S[b], self.field(b), w)
            del w
            acc &= self.occ[b]
            if self.sc:
                acc &= self.parity == c
            self.S[b] = torch.where(acc, new, self.S[b])
            n_acc += int(acc.sum())
        self.t += 1
        return n_acc

    def observables(self):
        m, pe2, sh = [0.0] * 3, 0.0, 0.0
        for b, S in enumerate(self.S):
            m = [m[a] + float(S[a].sum()) for a in range(3)]
            pe2 += float(((S[0] * self.e[0] + S[1] * self.e[1] + S[2] * self.e[2]) ** 2).sum())
            sh += 0.5 * float((S * self.field(b)).sum())
        m = [v / self.N for v in m]
        ex, an = -self.r["J"] * sh, -self.r["K"] * pe2
        return [*m, math.sqrt(sum(v * v for v in m)), ex + an, ex, an]

    def block_step(self, n, step):
        N = self.Lx * self.Ly * self.Lz
        k = torch.arange(-(-N // n), device=self.s[0].device)
        w = _words(k, self.r["replica_id"], step, 3, self.seed)
        s = k * n + ((w[3] * torch.clamp(N - k * n, max=n)) >> 32)
        S, h = self.S[0].reshape(3, -1), self.field(0).reshape(3, -1)
        new, acc = self.attempt(S[:, s], h[:, s], w)
        acc &= self.occ[0].reshape(-1)[s]
        S = S.clone()
        S[:, s[acc]] = new[:, acc]
        self.S[0] = S.view_as(self.S[0])

    def planes(self):
        """The library's colour-major layout."""
        out = []
        for a in range(3):
            if self.sc:
                odd = (self.parity[..., ::2]).reshape(-1).bool()  # parity of the even columns
                pair = self.S[0][a].reshape(-1, 2)
                out.append(torch.cat([torch.where(odd, pair[:, 1], pair[:, 0]),
                                      torch.where(odd, pair[:, 0], pair[:, 1])]))
            else:
                out.append(torch.cat([S[a].reshape(-1) for S in self.S]))
        return out

    def natural(self):
        return [torch.stack([S[a].reshape(-1) for S in self.S], 1).reshape(-1) for a in range(3)]


def exact(case, seed):
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    R = [_Exact(r, seed, dev) for r in _replicas(case)]
    cat = lambda planes: (list(planes[0]) if len(planes) == 1  # noqa: E731
                          else [torch.cat([p[a] for p in planes]) for a in range(3)])
    if case["do"] == "chain":
        rec = np.zeros((1, case["m"], len(R), 10))
        for i, x in enumerate(R):
            for _ in range(case["n"]):
                x.sweep()
            for j in range(case["m"]):
                n_acc = x.sweep()
                if case["api"] == "schedule" or j == case["m"] - 1:
                    o = x.observables()
                    rec[0, j, i] = [x.t, n_acc, *o, x.N]
        spins = cat([x.planes() for x in R])
        if case["api"] == "schedule":
            return {"records": rec, "spins": spins}
        last = rec[0, -1]
        return {"observables": np.concatenate([last[:, 2:9], last[:, 1:2]], 1), "spins": spins}
    if case["do"] == "exchange":
        T = [x.T for x in R]
        at = list(range(len(R)))
        for rnd in range(case["n"]):
            for x in R:
                for _ in range(case["m"]):
                    x.sweep()
            for k in range(rnd % 2, len(R) - 1, 2):
                Ei, Ej = R[at[k]].observables()[4], R[at[k + 1]].observables()[4]
                delta = (1.0 / T[k] - 1.0 / T[k + 1]) * (Ei - Ej)
                w = _words(torch.tensor([k]), 0, R[0].t, 2, seed)[0]
                if delta >= 0 or float(_u(w)[0]) < math.exp(delta):
                    at[k], at[k + 1] = at[k + 1], at[k]
            for k, i in enumerate(at):
                R[i].T = T[k]
        return {"slots": None, "accepted": None, "spins": cat([x.planes() for x in R])}
    if case["do"] == "block":
        for step in range(case["m"]):
            R[0].block_step(case["n"], step)
        return {"counts": None, "spins": R[0].planes()}
    return {"observables": np.array([R[0].observables()]), "natural": R[0].natural(),
            "spins": R[0].planes()}
