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
    a, b = _pair(M, name)
    for r, L in enumerate(CASES[name][1]):
        t = a.team(r)
        # a team's planes are the replica's
        assert t["workgroups"] >= 1
        assert (t["workgroups"] - 1) * t["planes"] + t["last_planes"] == L[2]
        assert 1 <= t["last_planes"] <= t["planes"]
        assert b.team(r)["workgroups"] == 0
    assert max(a.team(r)["workgroups"] for r in range(a.n_reps)) > 1


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
    single plane), of two members and of one, on periodic and open z."""
    seen = set()
    groups = [[(24, 24, lz)] * 11 for lz in (18, 26, 28, 30)]
    groups += [[(24, 24, lz)] * 20 for lz in (22, 26)]
    groups += [[(24, 24, 24), (6, 4, 2), (8, 8, 40)], [(40, 40, 2)] * 3, [(16, 16, 61)] * 16]
    for Ls in groups:
        mask = 7 if all(L[2] % 2 == 0 for L in Ls) else 3
        reps = [M.Replica(kind="sc", L=L, periodic_mask=mask, K=0.15, T=0.8 + 0.1 * r, replica_id=r)
                for r, L in enumerate(Ls)]
        a = M.Simulation(reps, precision="f32", seed=29)
        b = M.Simulation(reps, precision="f32", seed=29)
        b.set_tile(16, 16, 2, kernel=0)
        for r in range(len(Ls)):
            t = a.team(r)
            seen.add("one member" if t["workgroups"] == 1 else "two" if t["workgroups"] == 2 else "more")
            if t["workgroups"] > 1:
                seen.add("one plane" if t["planes"] == 1 else "planes")
                if t["last_planes"] < t["planes"]:
                    seen.add("short last")
                    if t["last_planes"] == 1:
                        seen.add("last of one plane")
        for s in (a, b):
            s.sweep(2, measure=True)
            s.sweep(2)
            s.sweep(1, measure=True)
        _same_spins(a, b)
        _same_obs(a.observables(), b.observables())
    assert seen == {"one member", "two", "more", "one plane", "planes", "short last",
                    "last of one plane"}
