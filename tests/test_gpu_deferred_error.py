"""A persistent launch that gave up (its wait budget set to zero from the host; it
ends normally) is reported by the next synchronising call, whichever that is, once,
before anyone takes its incomplete spins for a result."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    from paper_2106_11286_amd import mcheis

    return mcheis


@pytest.mark.parametrize("call", ["to_natural", "from_natural", "block_counts"])
def test_next_call_reports_it(M, call):
    reps = [M.Replica(kind="sc", L=L, K=0.1, T=0.8 + 0.3 * r, replica_id=r)
            for r, L in enumerate([(16, 16, 16), (24, 24, 24)])]
    sim = M.Simulation(reps, precision="f32", seed=5)
    spins = sim.to_natural(0)
    sim.block_steps(8, 0, 1)
    calls = {"to_natural": lambda: sim.to_natural(0),
             "from_natural": lambda: sim.from_natural(0, spins), "block_counts": sim.block_counts}
    sim.set_watchdog(0)
    sim.sweep(40, persistent=True)
    with pytest.raises(M.MCError) as ei:
        calls[call]()
    assert ei.value.status == -4 and "persistent" in str(ei.value)
    calls[call]()
    sim.set_watchdog(1 << 24)
    sim.sweep(2, persistent=True)
    calls[call]()
    sim.synchronize_checked()
