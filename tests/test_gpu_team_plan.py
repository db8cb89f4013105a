"""The handles that the team tests compare do run by teams, and their plans cover
the shapes a team can take (read from mc_get_team, not assumed)."""
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
def test_compared_handles(M, name):
    """Bitwise on calls of at least as many sweeps as the teams take, and on ones
    of fewer; only a lattice of two wide planes is left to the plain kernels."""
    a, b = _pair(M, name)
    plain, measured = a.team()["from"]
    if name == "two-planes":
        assert a.team()["workgroups"] == 0
        return
    for r, L in enumerate(CASES[name][1]):
        t = a.team(r)
        # a team's planes are the replica's
        assert t["workgroups"] >= 1
        assert (t["workgroups"] - 1) * t["planes"] + t["last_planes"] == L[2]
        assert 1 <= t["last_planes"] <= t["planes"]
        assert b.team(r)["workgroups"] == 0
    assert max(a.team(r)["workgroups"] for r in range(a.n_reps)) > 1
    assert min(plain, measured) <= 64
    for n, measure in ((64, True), (64, False), (min(measured, 64), True), (1, True),
                       (min(plain, 64), False), (1, False), (130, True)):
        for s in (a, b):
            s.sweep(n, measure=measure)
    _same_spins(a, b)
    _same_obs(a.observables(), b.observables())


def test_calls_that_the_teams_take(M):
    """The number of sweeps from which a call runs by teams, seen by the launches
    that a zero wait budget makes them do again: eager calls, schedules, timed."""
    a = M.Simulation([M.Replica(kind="sc", L=(24, 24, 24), K=0.1, T=1.0)], precision="f32", seed=2)
    b = M.Simulation([M.Replica(kind="sc", L=(24, 24, 24), K=0.1, T=1.0)], precision="f32", seed=2)
    b.set_tile(16, 16, 2, kernel=0)
    plain, measured = a.team()["from"]
    # one sweep costs two or three plain launches less than filling the planes
    assert 1 < plain <= 64 and 1 < measured <= 64
    a.set_watchdog(0)
    count = 0
    for n, measure in ((plain - 1, False), (plain, False), (measured - 1, True), (measured, True)):
        a.sweep(n, measure=measure)
        b.sweep(n, measure=measure)
        count += n >= (measured if measure else plain)
        assert a.team()["redone"] == count
    a.sweep_timed(plain - 1)
    a.sweep_timed(plain)
    b.sweep(2 * plain - 1)
    assert a.team()["redone"] == count + 1
    # chunks of up to 64 sweeps: 64 + 1 to equilibrate, 64 + 1 measured
    ra, rb = (s.run_schedule([1.2], n_equil=65, n_meas=65) for s in (a, b))
    assert a.team()["redone"] == count + 3
    assert (ra[..., 0:2] == rb[..., 0:2]).all()
    _same_spins(a, b)


@pytest.mark.parametrize("spare", [None, 0, 1 << 20, 16 << 20])
def test_workspaces(M, spare):
    """Teams with the default scratch, without room in it and with room, after a
    tile change and back, and after a tune whose choice they are."""
    import torch

    reps = [M.Replica(kind="sc", L=(24, 24, 24), K=0.1, T=1.0 + 0.1 * r, replica_id=r)
            for r in range(5)]
    scratch = None
    if spare is not None:
        scratch = torch.full((M.required_scratch(reps) + spare,), 255, dtype=torch.uint8,
                             device="cuda")
    a = M.Simulation(reps, precision="f32", seed=9, scratch=scratch)
    team = a.team()
    assert team["workgroups"] > 1
    tile = a.get_tile()
    a.set_tile(256, 2, 4, kernel=2)
    assert a.team()["workgroups"] == 0
    a.set_tile(*tile[1:4], kernel=tile[0])
    assert a.team() == team
    a.autotune(trial_sweeps=1, measure=True)
    assert a.team()["workgroups"] in (0, team["workgroups"])
    if a.team()["workgroups"]:
        assert a.get_tile()[:4] == tile[:4]


def test_plans_of_every_shape(M):
    """Teams of one plane each, of several, with a shorter last member (down to a
    single plane) and of one member beside others, on periodic and open z."""
    seen = set()
    groups = [[(24, 24, lz)] * 11 for lz in (18, 26, 28, 30)]
    groups += [[(24, 24, lz)] * 20 for lz in (22, 26)]
    groups += [[(24, 24, 24), (6, 4, 2), (8, 8, 40)], [(16, 16, 61)] * 16]
    for Ls in groups:
        mask = 7 if all(L[2] % 2 == 0 for L in Ls) else 3
        reps = [M.Replica(kind="sc", L=L, periodic_mask=mask, K=0.15, T=0.8 + 0.1 * r, replica_id=r)
                for r, L in enumerate(Ls)]
        a = M.Simulation(reps, precision="f32", seed=29)
        b = M.Simulation(reps, precision="f32", seed=29)
        b.set_tile(16, 16, 2, kernel=0)
        for r in range(len(Ls)):
            t = a.team(r)
            seen.add("one member" if t["workgroups"] == 1 else "more")
            if t["workgroups"] > 1:
                seen.add("one plane" if t["planes"] == 1 else "planes")
                if t["last_planes"] < t["planes"]:
                    seen.add("short last")
                    if t["last_planes"] == 1:
                        seen.add("last of one plane")
        for s in (a, b):
            s.sweep(40, measure=True)
            s.sweep(50)
            s.sweep(20, measure=True)
        _same_spins(a, b)
        _same_obs(a.observables(), b.observables())
    assert seen == {"one member", "more", "one plane", "planes", "short last", "last of one plane"}
