"""Team sweeps whose waits give up: every workgroup leaves, one per replica does
the launch again, and nothing is lost.  A wait budget of zero, set from the host,
makes every launch of a team end that way."""
import numpy as np
import pytest

from test_gpu_team import CASES, _pair, _same_obs, _same_spins

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    from paper_2106_11286_amd import mcheis

    return mcheis


@pytest.mark.parametrize("name", list(CASES))
def test_given_up_sweeps_are_bitwise(M, name):
    a, b = _pair(M, name)
    teams = sum(a.team(r)["workgroups"] > 1 for r in range(a.n_reps))
    plain, measured = a.team()["from"]
    if teams == 0:
        pytest.skip("never swept by teams")
    assert a.team()["redone"] == 0
    # as many sweeps as the teams take, and more (calls that they never take: one)
    calls = [(min(n + k, 64) if n <= 64 else 1, m) for k in (0, 3)
             for m, n in ((True, measured), (False, plain))]
    by_teams = 2 * (measured <= 64) + 2 * (plain <= 64)
    assert by_teams > 0
    launches = 0
    for spins in (0, 1 << 24, 0):
        a.set_watchdog(spins)
        for n, measure in calls:
            a.sweep(n, measure=measure)
            b.sweep(n, measure=measure)
        a.synchronize_checked()
        launches += 0 if spins else by_teams
        assert a.team()["redone"] == launches * teams
        _same_spins(a, b)
        _same_obs(a.observables(), b.observables())
        for s in (a, b):
            s.sweep(1, measure=True)
        launches += (spins == 0) * (measured == 1)
    assert [o["n_sites"] for o in a.measure_state()] == a.n_occ


@pytest.mark.parametrize("spins", [0, 3])
def test_given_up_schedules_and_exchange(M, spins):
    """Schedules (more sweeps than a launch takes) and replica exchange, which
    read the records of launches that were done again; with a small budget some
    launches are and some are not."""
    reps = [M.Replica(kind="sc", L=(16, 16, 16), K=0.05, T=1.3 + 0.05 * r, replica_id=r)
            for r in range(6)]
    a = M.Simulation(reps, precision="f64", seed=3)
    b = M.Simulation(reps, precision="f64", seed=3)
    b.set_tile(16, 16, 2, kernel=0)
    a.set_watchdog(spins)
    assert a.team()["workgroups"] > 1
    ra, rb = (s.run_schedule([1.1, 1.4], n_equil=70, n_meas=70) for s in (a, b))
    assert np.array_equal(ra[..., 0:2], rb[..., 0:2])
    assert np.max(np.abs(ra[..., 2:5] - rb[..., 2:5])) <= 1e-12
    for s in (a, b):
        s.exchange_init()
        s.exchange_sweep(5, 3)
    assert a.exchange_state() == b.exchange_state()
    _same_spins(a, b)
    if spins == 0:
        assert a.team()["redone"] > 0


def test_given_up_beside_other_handles(M):
    """Handles side by side, one of them redoing every launch."""
    sims = [_pair(M, "uneven-batch", seed=s) for s in range(4)]
    sims[1][0].set_watchdog(0)
    for _ in range(4):
        for a, _b in sims:
            a.sweep(20, measure=True)
    for a, b in sims:
        b.sweep(80, measure=True)
        _same_spins(a, b)
        _same_obs(a.observables(), b.observables())
    assert sims[1][0].team()["redone"] > 0


def test_team_query(M):
    a, b = _pair(M, "open-odd-edges")
    assert a.team()["workgroups"] > 1 and b.team()["workgroups"] == 0
    with pytest.raises(M.MCError):
        a.team(1)
    # the spins stay those of the handle's own tile after the query
    a.sweep(2)
    b.sweep(2)
    _same_spins(a, b)
