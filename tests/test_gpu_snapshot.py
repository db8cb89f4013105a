"""Layout conversion and from-scratch observables at the sizes where their
vector widths, workgroup counts and edges change, against numpy."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

BASIS = {"sc": [(0, 0, 0)], "bcc": [(0, 0, 0), (1, 1, 1)],
         "fcc": [(0, 0, 0), (1, 1, 0), (1, 0, 1), (0, 1, 1)]}
FWD = {"sc": [(2, 0, 0), (0, 2, 0), (0, 0, 2)],
       "bcc": [(1, 1, 1), (1, 1, -1), (1, -1, 1), (1, -1, -1)],
       "fcc": [(1, 1, 0), (1, -1, 0), (1, 0, 1), (1, 0, -1), (0, 1, 1), (0, 1, -1)]}

CASES = [("sc", (50, 37, 23), 0, 0.0),    # odd colour plane: one column per thread
         ("sc", (6, 5, 3), 1, 0.0),       # rows shorter than a vector of columns
         ("sc", (2, 2, 4), 7, 0.0),       # periodic lengths of two: every bond twice
         ("sc", (64, 32, 16), 7, 0.0),    # a multiple of eight workgroups
         ("sc", (40, 38, 26), 0, 11.3),   # sphere
         ("sc", (34, 30, 28), 6, 0.0),    # one open axis
         ("bcc", (5, 3, 1), 7, 0.0),      # a periodic length of one
         ("bcc", (21, 19, 17), 2, 0.0),
         ("bcc", (16, 16, 16), 0, 7.1),
         ("fcc", (9, 7, 5), 7, 0.0),
         ("fcc", (16, 15, 14), 5, 0.0),
         ("fcc", (18, 18, 18), 0, 8.2)]


def _grid(kind, L):
    z, y, x = np.meshgrid(*(np.arange(n) for n in (L[2], L[1], L[0])), indexing="ij")
    nb = len(BASIS[kind])
    out = []
    for a, c in enumerate((x, y, z)):
        off = np.array([b[a] for b in BASIS[kind]])
        out.append((2 * c.reshape(-1, 1) + off).reshape(-1))  # half cells, canonical order
    return out, nb


def _expected(rep, S):
    """M sums, E_exch, E_anis and the number of occupied sites, bond by bond."""
    kind, L = rep.kind, rep.L
    q, nb = _grid(kind, L)
    occ = np.ones(q[0].size, bool)
    if rep.sphere_radius > 0:
        occ = sum((q[a] - L[a]) ** 2 for a in range(3)) <= 4 * rep.sphere_radius ** 2
    table = {p: b for b, p in enumerate(BASIS[kind])}
    bond = 0.0
    for d in FWD[kind]:
        ok = occ.copy()
        n = []
        for a in range(3):
            v = q[a] + d[a]
            out = (v < 0) | (v >= 2 * L[a])
            if not rep.periodic_mask >> a & 1:
                ok &= ~out
            n.append(v % (2 * L[a]))
        b2 = np.array([[[table.get((i, j, k), 0) for k in (0, 1)] for j in (0, 1)]
                       for i in (0, 1)])[n[0] & 1, n[1] & 1, n[2] & 1]
        j = (((n[2] >> 1) * L[1] + (n[1] >> 1)) * L[0] + (n[0] >> 1)) * nb + b2
        ok &= occ[j]
        bond += sum((S[a] * S[a][j])[ok].sum() for a in range(3))
    e = np.array(rep.e) / np.linalg.norm(rep.e)
    pe = sum(S[a] * e[a] for a in range(3))
    return ([S[a][occ].sum() for a in range(3)], -rep.J * bond, -rep.K * (pe[occ] ** 2).sum(),
            int(occ.sum()))


def _packed_index(kind, L):
    n = L[0] * L[1] * L[2]
    if kind == "sc":
        z, y, x = np.meshgrid(*(np.arange(m) for m in (L[2], L[1], L[0])), indexing="ij")
        c = (x + y + z) & 1
        return (c * (n // 2) + ((z * L[1] + y) * L[0] + x) // 2).reshape(-1)
    nb = len(BASIS[kind])
    cell = np.arange(n)
    return np.stack([b * n + cell for b in range(nb)], 1).reshape(-1)


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_snapshot(case, prec):
    from paper_2106_11286_amd import mcheis as M

    kind, L, mask, R = CASES[case]
    rep = M.Replica(kind=kind, L=L, periodic_mask=mask, sphere_radius=R, J=1.0, K=0.3,
                    e=(0.3, 0.2, 0.9), T=1.0)
    sim = M.Simulation([rep], precision=prec, seed=case)
    # to natural order: the documented layout, bit for bit
    packed = [t.cpu().numpy() for t in sim.state_spins(0)]
    nat = sim.to_natural(0)
    idx = _packed_index(kind, L)
    for p, t in zip(packed, nat):
        assert np.array_equal(p[idx], t.cpu().numpy())
    # observables (sums of at most 2e4 unit terms in FP64, another order)
    S = [t.double().cpu().numpy() for t in nat]
    m, ex, an, n = _expected(rep, S)
    o = sim.measure_state()[0]
    r = M.measure_buffers(rep, prec, *sim.state_spins(0))
    assert o["n_sites"] == n and r["n_sites"] == n
    tol = 1e-14 * 12 * n
    assert np.max(np.abs(o["M"] * n - m)) <= tol
    assert abs(o["E_exch"] - ex) <= tol and abs(o["E_anis"] - an) <= tol
    assert o["E_exch"] == r["E_exch"] and o["E_anis"] == r["E_anis"]
    # and back
    rng = np.random.default_rng(case)
    new = [rng.normal(size=S[0].size).astype(packed[0].dtype) for _ in range(3)]
    sim.from_natural(0, new)
    for p, t in zip(sim.state_spins(0), new):
        assert np.array_equal(p.cpu().numpy()[idx], t)
