"""The sweep counter of the pass kernels over every way to enqueue sweeps: several
together, one at a time, measured or not, timed, as schedules (captured graphs),
after the counter is set."""
import numpy as np
import pytest

from test_gpu_team import _same_obs, _same_spins

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    from paper_2106_11286_amd import mcheis

    return mcheis


@pytest.mark.parametrize("kind,L,tile", [("sc", (20, 12, 10), (256, 2, 2, 2)),
                                         ("bcc", (10, 9, 8), (64, 4, 2, 6)),
                                         ("fcc", (10, 6, 8), (64, 1, 2, 7))])
def test_counter_over_every_route(M, kind, L, tile):
    reps = [M.Replica(kind=kind, L=L, K=0.1, T=1.0 + 0.2 * r, replica_id=r) for r in range(2)]
    a = M.Simulation(reps, precision="f64", seed=13)
    b = M.Simulation(reps, precision="f64", seed=13)
    a.set_tile(*tile[:3], kernel=tile[3])
    b.set_tile(8, 8, 3, kernel=0)

    def same(t):
        for _ in range(t - b.get_sweep() - 1):
            b.sweep(1)
        b.sweep(1, measure=True)
        assert a.get_sweep() == t == b.get_sweep()
        _same_spins(a, b)

    t = 0
    for n, measure in ((1, True), (3, True), (2, False), (5, True), (1, False), (4, True)):
        a.sweep(n, measure=measure)
        t += n
        same(t)
        if measure:
            _same_obs(a.observables(), b.observables())
            assert all(o["sweep"] == t for o in a.observables())
    a.sweep_timed(3, measure=True)
    t += 3
    same(t)
    _same_obs(a.observables(), b.observables())
    for k in range(3):  # the graphs of the first round replayed, eager sweeps between
        rec = a.run_schedule([1.1], n_equil=5, n_meas=3)
        b.set_temperatures([1.1, 1.1])
        assert np.array_equal(rec[0, :, 0, 0], t + 5 + 1 + np.arange(3))
        t += 8
        same(t)
        a.sweep(2)
        t += 2
        same(t)
    for s in (a, b):
        s.set_sweep(7)
    a.sweep(3, measure=True)
    same(10)
    _same_obs(a.observables(), b.observables())
