"""Team sweeps and the autotuner: its cache says whether the choice ran by teams,
and timing the teams leaves the chain where it was."""
import pytest

from test_gpu_team import _same_obs, _same_spins

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    from paper_2106_11286_amd import mcheis

    return mcheis


LATTICES = {"lds": ("sc", (16, 16, 16), "f64"), "pass": ("sc", (24, 24, 24), "f32"),
            "bcc": ("bcc", (12, 12, 12), "f32")}


def _sim(M, name):
    kind, L, prec = LATTICES[name]
    return M.Simulation([M.Replica(kind=kind, L=L, K=0.1, T=1.2)], precision=prec, seed=4)


@pytest.mark.parametrize("tune_launch", [False, True])
@pytest.mark.parametrize("name", list(LATTICES))
def test_cache_keeps_the_teams_choice(M, tmp_path, name, tune_launch):
    cache = tmp_path / "tune.txt"
    a = _sim(M, name)
    team = a.team()
    assert team["workgroups"] > 1
    default = a.get_tile()[:4]
    tile = a.autotune(trial_sweeps=2, measure=True, tune_launch=tune_launch, cache_path=str(cache))
    fields = cache.read_text().split()
    assert len(fields) == 8 and fields[7] == str(int(a.team()["workgroups"] > 0))
    if fields[7] == "1":
        assert tuple(tile) == default

    def hit(text):
        cache.write_text(text + "\n")
        s = _sim(M, name)
        s.autotune(trial_sweeps=2, measure=True, tune_launch=tune_launch, cache_path=str(cache))
        assert s.get_sweep() == 0  # no trials
        return s

    # the default tile: as the entry says, without the field not by teams
    line = " ".join([fields[0]] + [str(v) for v in default] + ["0.01"])
    with_teams, without, old = hit(line + " 0 1"), hit(line + " 0 0"), hit(line)
    assert with_teams.team() == team
    assert without.team()["workgroups"] == 0 and old.team()["workgroups"] == 0
    # the entry written by the run itself
    again = hit(" ".join(fields))
    assert again.get_tile()[:4] == a.get_tile()[:4]
    assert again.team()["workgroups"] == a.team()["workgroups"]
    # another tile is never swept by teams
    other = hit(" ".join([fields[0], "0", "8", "8", "2", "0.01", "0", "1"]))
    assert other.get_tile()[:4] == (0, 8, 8, 2) and other.team()["workgroups"] == 0
    for s in (with_teams, without, old, again, other):
        s.sweep(12, measure=True)
        _same_spins(s, with_teams)
        _same_obs(s.observables(), with_teams.observables())


@pytest.mark.parametrize("name", list(LATTICES))
def test_timing_the_teams_takes_no_step(M, name):
    """The state after the trials is that of as many plain sweeps, the counter
    that of the plain candidates: one sweep and the trial sweeps of each."""
    a, b = _sim(M, name), _sim(M, name)
    a.autotune(trial_sweeps=3, measure=True)
    t = a.get_sweep()
    assert t > 0 and t % 4 == 0
    b.set_tile(8, 8, 3, kernel=0)
    b.sweep(t)
    _same_spins(a, b)
    for s in (a, b):
        s.sweep(2, measure=True)
    _same_obs(a.observables(), b.observables())
    # persistent tuning has no teams
    c = _sim(M, name)
    c.autotune(trial_sweeps=1, persistent=True)
    assert c.team()["workgroups"] == 0
