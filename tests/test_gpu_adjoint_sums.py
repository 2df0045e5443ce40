"""The sums of the 3D FP32 step adjoint (lamE, lamB of a tile) against the
global-memory path: full tiles, adjoints near both ends of the FP32 range, and
adjoints that are infinite or NaN."""
import numpy as np
import pytest

from paper_1310_0930_amd import inputs as I

from _parity import inputs_for
from test_gpu_adjoint import _sim, _t

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _both(order, ppc, amp, poison=None):
    """(lamE, lamB, lamX, lamU) out of LDS tiles and in global memory."""
    from paper_1310_0930_amd import pic as P
    w = I.Workload("adjs", 3, (16, 12, 9), (0.2, 0.25, 0.2), order, ppc, 0.3, 1, bc=(0, 1, 0),
                   ramp_cells=4.0, seed=I.SEED_BASE + 170 + order)
    pl, E, B = inputs_for(w)
    sim = _sim(w, 4)
    sim.load(pl, E, B, with_id=True)
    sim.sort()
    rng = np.random.default_rng(71 + order + ppc)
    lam = [_t(amp * rng.normal(size=s), sim) for s in ((3, sim.ncell),) * 3 + ((3, sim.np),) * 2]
    if poison is not None:
        lam[4][1, sim.np // 2] = poison
    out = []
    for ws in (sim.ws, torch.zeros_like(sim.ws)):
        LE, LB, LJ, LX, LU = (t.clone() for t in lam)
        P.pic_push_deposit_adjoint(sim.ctx, P.particles_struct(sim.np, sim.cell, sim.off, sim.u, sim.q),
                                   P.fields_struct(sim.E, sim.B), P.fields_struct(LE, LB, LJ),
                                   P.particles_struct(sim.np, None, LX, LU), ws.data_ptr(), sim.stream)
        torch.cuda.synchronize()
        out.append([t.double().cpu().numpy() for t in (LE, LB, LX, LU)])
    return out


# A node sums at most (order + 1)^3 products of each of some 20 particles a
# cell: at 24 bits 125 x 20 x 2^-24 = 1.5e-4 of the largest, when every
# rounding falls the same way.
TOL = 2e-4


@pytest.mark.parametrize("order,ppc,amp", [(1, 4, 1.0), (2, 9, 1.0), (2, 20, 1.0), (3, 20, 1e-25),
                                           (2, 4, 1e25), (4, 20, 1.0)])
def test_fixed_point_sums_equal_global_memory(order, ppc, amp):
    tiled, glob = _both(order, ppc, amp)
    for a, b in zip(tiled, glob):
        assert np.abs(a - b).max() <= TOL * np.abs(b).max()


@pytest.mark.parametrize("poison", [float("nan"), float("inf")])
@pytest.mark.parametrize("order", [1, 2, 3, 4])
def test_non_finite_adjoints_reach_the_same_samples(order, poison):
    tiled, glob = _both(order, 4, 1.0, poison)
    for a, b in zip(tiled, glob):
        bad = ~np.isfinite(b)
        assert np.array_equal(~np.isfinite(a), bad)
        assert np.abs(a - b)[~bad].max() <= TOL * np.abs(b[~bad]).max()
    assert not np.isfinite(tiled[0]).all()
