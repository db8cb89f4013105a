"""The default tile of bcc / fcc lattices with odd rows: the basis strip kernel
from 33 cells per row on, the tile kernel below; either gives the spins and the
accepted counts of the tile kernel on a plain tile."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("kind", ["bcc", "fcc"])
@pytest.mark.parametrize("Ls,R,kernel", [([(31, 40, 60)], 0.0, 0), ([(33, 37, 47)], 0.0, 6),
                                         ([(65, 41, 23)], 0.0, 6), ([(129, 18, 25)], 0.0, 6),
                                         ([(47, 45, 41)], 21.0, 6),
                                         ([(33, 40, 40), (64, 31, 21)], 0.0, 6),
                                         ([(33, 40, 40), (32, 41, 41)], 0.0, 0)])
def test_odd_rows(prec, kind, Ls, R, kernel):
    import torch

    from paper_2106_11286_amd import mcheis as M

    reps = [M.Replica(kind=kind, L=L, K=0.1, e=(0.0, 0.6, 0.8), T=1.1 + r, replica_id=r,
                      sphere_radius=R, periodic_mask=0 if R else 5 + r)
            for r, L in enumerate(Ls)]

    def run(tile):
        sim = M.Simulation(reps, precision=prec, seed=3,
                           scratch=torch.empty(64 << 20, dtype=torch.uint8, device="cuda"))
        if tile:
            sim.set_tile(*tile, kernel=0)
        else:
            sim.set_tile(*sim.get_tile()[1:4], kernel=sim.get_tile()[0])
            assert sim.get_tile()[0] == kernel
        sim.sweep(2)
        sim.sweep(1, measure=True)
        return [[t.cpu().numpy() for t in sim.to_natural(r)] for r in range(len(reps))], \
            [o["n_accepted"] for o in sim.observables()]

    got, ref = run(None), run((16, 16, 2))
    assert got[1] == ref[1]
    for a, b in zip(got[0], ref[0]):
        for x, y in zip(a, b):
            assert np.array_equal(x, y)
