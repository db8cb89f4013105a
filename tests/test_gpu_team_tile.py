"""Team sweeps beside mc_set_tile, mc_get_tile and mc_sweep_timed."""
import pytest

from test_gpu_team import _same_obs, _same_spins

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    from paper_2106_11286_amd import mcheis

    return mcheis


# whole lattice in LDS by default; a pass kernel by default; basis lattice
LATTICES = {"lds": ("sc", (16, 16, 16), "f64"), "pass": ("sc", (24, 24, 24), "f32"),
            "fcc": ("fcc", (12, 12, 12), "f32")}


def _sims(M, name, n=2):
    kind, L, prec = LATTICES[name]
    reps = [M.Replica(kind=kind, L=L, K=0.1, T=1.0 + 0.2 * r, replica_id=r) for r in range(3)]
    return [M.Simulation(reps, precision=prec, seed=31) for _ in range(n)]


@pytest.mark.parametrize("name", list(LATTICES))
def test_default_tile_brings_the_teams_back(M, name):
    a, b = _sims(M, name)
    k, tx, ty, zc = a.get_tile()[:4]
    team = a.team()
    assert team["workgroups"] > 1
    b.set_tile(16, 16, 2, kernel=0)
    assert b.team()["workgroups"] == 0
    a.set_tile(tx, ty, zc, kernel=k)  # as it reads
    assert a.team() == team
    a.set_tile(8, 8, 3, kernel=0)
    assert a.team()["workgroups"] == 0
    for s in (a, b):
        s.sweep(2, measure=True)
    a.set_tile(tx, ty, zc, kernel=k)
    assert a.team() == team and a.get_tile()[:4] == (k, tx, ty, zc)
    for s in (a, b):
        s.sweep(9, measure=True)
    _same_spins(a, b)
    _same_obs(a.observables(), b.observables())


@pytest.mark.parametrize("name", list(LATTICES))
def test_timed_sweeps_run_the_teams(M, name):
    """mc_sweep_timed times what mc_sweep runs: with no wait budget every launch
    of a team is done again, and counted."""
    a, b = _sims(M, name)
    for measure in (False, True):
        per_colour, total = a.sweep_timed(70, measure=measure)
        assert 0 < per_colour < total
        b.sweep(70, measure=measure)
    a.set_watchdog(0)
    before = a.team()["redone"]
    a.sweep_timed(9)
    b.sweep(9)
    assert a.team()["redone"] == before + a.n_reps
    _same_spins(a, b)
    _same_obs(a.observables(), b.observables())
