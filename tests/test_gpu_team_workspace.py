"""The workspace of team sweeps beside the autotuner's larger scratch layouts."""
import pytest

from test_gpu_team import _same_obs, _same_spins

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    from paper_2106_11286_amd import mcheis

    return mcheis


# whole lattices in LDS by default, whose autotuner candidates need more scratch
# than the default layout (long wires, batches of small cubes)
LDS_DEFAULTS = {
    "wires": [(8, 8, 100)] * 12,
    "long-wires": [(4, 4, 400)] * 8,
    "cubes": [(20, 20, 20)] * 22,
}


@pytest.mark.parametrize("spare", [0, 32 << 20])
@pytest.mark.parametrize("name", list(LDS_DEFAULTS))
def test_team_after_autotune_of_an_lds_default(M, name, spare):
    """After the autotuner's larger layouts, measurements, block steps and
    measured sweeps leave the teams' state alone."""
    import torch

    reps = [M.Replica(kind="sc", L=L, K=0.1, T=0.9 + 0.1 * r, replica_id=r)
            for r, L in enumerate(LDS_DEFAULTS[name])]
    scratch = None
    if spare:
        scratch = torch.empty(M.required_scratch(reps) + spare, dtype=torch.uint8, device="cuda")
    a = M.Simulation(reps, precision="f32", seed=17, scratch=scratch)
    assert a.get_tile()[0] == 3
    a.autotune(trial_sweeps=1, measure=True)
    t = a.get_sweep()
    b = M.Simulation(reps, precision="f32", seed=17)
    b.set_tile(8, 8, 4, kernel=0)
    b.sweep(t, measure=True)
    for _ in range(2):
        _same_obs(a.measure_state(), b.measure_state())
        for s in (a, b):
            s.block_steps(8, 0, 2)
            s.sweep(12, measure=True)
        _same_spins(a, b)
        _same_obs(a.observables(), b.observables())
