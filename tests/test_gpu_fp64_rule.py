"""FP64 decisions where the FP32 exponential alone could not give them: the
whole range of beta*dH, from greedy-like temperatures (the FP32 exponential
overflows or vanishes) to hot ones (every proposal near the acceptance edge)."""
import numpy as np
import pytest

from oracle import oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [0.01, 0.3, 4.0, 1e4])
def test_fp64_decisions_equal_the_oracles(T):
    """One sweep of 2.6e5 sites: accepted moves equal to the oracle's and spins
    to 1e-15 (a few rounding errors of unit components; a differing decision
    would move a spin by O(1))."""
    from paper_2106_11286_amd import mcheis as M

    L = 64
    rep = M.Replica(kind="sc", L=(L, L, L), J=1.0, K=0.3, e=(0.6, 0.0, 0.8), T=T)
    sim = M.Simulation([rep], precision="f64", seed=17)
    geo = O.Lattice(O.SC, L)
    p = O.Params(J=1.0, K=0.3, e=(0.6, 0.0, 0.8), T=T, seed=17)
    s = O.init(geo, p)
    before = [a.copy() for a in s]
    ref = O.run(geo, p, 0, 1, s)
    sim.sweep(1, measure=True)
    o = sim.observables()[0]
    got = [a.cpu().numpy() for a in sim.to_natural(0)]
    assert o["n_accepted"] == int(ref[0, 5])
    assert max(np.abs(a - b).max() for a, b in zip(got, s)) <= 1e-15
    moved = sum(np.count_nonzero(a != b) for a, b in zip(got, before))
    assert (moved > 0) == (ref[0, 5] > 0)
