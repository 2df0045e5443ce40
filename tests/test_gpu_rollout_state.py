"""The state a rollout leaves in its simulation."""
import numpy as np
import pytest

from paper_1310_0930_amd import inputs as I

from _parity import inputs_for

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("steps,every", [(6, 10), (6, 6), (1, 5)])
def test_backward_of_one_segment_leaves_the_final_state(steps, every):
    """A rollout that fits one checkpoint segment is recomputed whole by its
    backward, after which the simulation is again where the forward left it
    (up to the order of the current's atomic additions): a diagnostic taken
    after the gradient is of the final state."""
    from paper_1310_0930_amd.adjoint import PicRollout, Runner
    lz = I.Laser(a0=2.0, omega0=6.0, waist=1.5, tau=0.5, x_center=1.5)
    w = I.Workload("rollstate", 2, (64, 24), (0.1, 0.2), 2, 4, 0.0, steps, bc=(0, 1), ramp_cells=10.0,
                   laser=lz, seed=I.SEED_BASE + 98)
    pl, E1, B1 = inputs_for(w)
    runner = Runner(w, real_bytes=8, checkpoint_every=every)
    runner.set_inputs(pl, E1 / lz.a0, B1 / lz.a0)
    a0 = torch.tensor(lz.a0, dtype=torch.float64, device="cuda", requires_grad=True)
    u0 = torch.from_numpy(pl.u).to("cuda", torch.float64).requires_grad_()
    E, B = PicRollout.apply(a0, u0, runner)
    s = runner.sim
    before = {k: getattr(s, k).clone() for k in ("E", "B", "J", "off", "u")}
    assert torch.equal(E.detach(), s.E) and torch.equal(B.detach(), s.B)
    torch.autograd.backward((E, B), (torch.ones_like(E), torch.ones_like(B)))
    for k, v in before.items():
        now = getattr(s, k)
        far = float((now - v).abs().max() / v.abs().max())
        print("rollout state", steps, every, k, far, flush=True)
        assert far <= 1e-9, k
