"""The second buffer sets are filled before the library may write them: with
torch's stream still busy when they are allocated, the sweeps that follow on
the library's own stream keep what they write."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_second_buffers_ready_before_use(prec):
    import torch

    from paper_2106_11286_amd import mcheis as M

    rep = M.Replica(kind="sc", L=(64, 32, 32), K=0.1, T=1.2)

    def sim():
        return M.Simulation([rep], precision=prec, seed=5,
                            scratch=torch.empty(16 << 20, dtype=torch.uint8, device="cuda"))

    ref = sim()
    ref.set_tile(64, 4, 8, kernel=0)
    ref.sweep(1)
    one = sim()
    busy = torch.empty(256 << 20, dtype=torch.float32, device="cuda")
    for k in range(100):  # some 20 ms on torch's stream
        busy.fill_(k)
    one.enable_fused()
    one.set_tile(256, 2, 16, kernel=9)
    one.sweep(1)
    torch.cuda.synchronize()
    for a, b in zip(one.state_spins(0), ref.state_spins(0)):
        assert torch.equal(a, b)
