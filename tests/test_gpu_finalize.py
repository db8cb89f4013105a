"""Records of measured sweeps where the reduction of the work items' sums
changes shape: one workgroup per replica, a few of them, all 32; uneven
batches; several calls in a row (the workgroups' count starts over each time)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# (kind, L of the replicas, tile, kernel): work items times colours per replica
CASES = [("sc", [(64, 32, 16)], (64, 2, 16), 1),            # 32 slots: one workgroup
         ("sc", [(64, 64, 16)], (64, 2, 2), 1),             # 512: the most for one
         ("sc", [(64, 64, 18)], (64, 2, 2), 1),             # 576: two
         ("sc", [(64, 128, 136)], (64, 1, 1), 1),           # 34816: 32, the most
         ("sc", [(64, 64, 32), (16, 8, 6), (64, 2, 2)], (64, 1, 1), 1),
         ("bcc", [(32, 40, 40)], (32, 1, 1), 0),
         ("fcc", [(16, 24, 20), (8, 3, 2)], (16, 1, 1), 0)]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_records_equal_the_state(case):
    import torch

    from paper_2106_11286_amd import mcheis as M

    kind, Ls, (tx, ty, zc), kernel = CASES[case]
    reps = [M.Replica(kind=kind, L=L, K=0.2, e=(0.1, 0.0, 1.0), T=1.0 + r, replica_id=r)
            for r, L in enumerate(Ls)]
    sim = M.Simulation(reps, precision="f64", seed=case,
                       scratch=torch.empty(64 << 20, dtype=torch.uint8, device="cuda"))
    sim.set_tile(tx, ty, zc, kernel=kernel)
    for n in (1, 2, 3):
        sim.sweep(n, measure=True)
        for o, s in zip(sim.observables(), sim.measure_state()):
            assert o["sweep"] == s["sweep"] and o["n_sites"] == s["n_sites"]
            # FP64 sums of N unit terms (12 N for the bonds) in another order
            tol = 12 * s["n_sites"] * 2.0 ** -52
            assert np.max(np.abs(o["M"] - s["M"])) * s["n_sites"] <= tol
            assert abs(o["E_exch"] - s["E_exch"]) <= tol
            assert abs(o["E_anis"] - s["E_anis"]) <= tol
    # graph-replayed records, with an eager sweep between the replays
    for _ in range(3):
        rec = sim.run_schedule([1.5], 0, 4)
        last = sim.measure_state()
        for r, s in enumerate(last):
            assert rec[0, -1, r, 0] == s["sweep"]
            assert abs(rec[0, -1, r, 6] - s["E"]) <= 24 * s["n_sites"] * 2.0 ** -52
        sim.sweep(1, measure=True)
