"""The transpose of the gather node by node, with adjoints that fall by many
decades inside a tile: FP32 against the same state in FP64."""
import numpy as np
import pytest

from paper_1310_0930_amd import inputs as I

from _parity import inputs_for
from test_gpu_adjoint import _sim, _t

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _lam_e(w, rb, pl, E, B, lam):
    from paper_1310_0930_amd import pic as P
    sim = _sim(w, rb)
    sim.load(pl, E, B, with_id=True)
    sim.sort()
    LE, LB, LJ = (torch.zeros_like(sim.E) for _ in range(3))
    LX = torch.zeros_like(sim.off)
    LU = _t(lam[:, sim.id.long().cpu().numpy()], sim)
    P.pic_push_deposit_adjoint(sim.ctx, P.particles_struct(sim.np, sim.cell, sim.off, sim.u, sim.q),
                               P.fields_struct(sim.E, sim.B), P.fields_struct(LE, LB, LJ),
                               P.particles_struct(sim.np, None, LX, LU), sim.ws.data_ptr(), sim.stream)
    torch.cuda.synchronize()
    return LE.double().cpu().numpy()


@pytest.mark.parametrize("decades", [0, 1, 2])
@pytest.mark.parametrize("dims,order", [(3, 1), (3, 2), (3, 3), (3, 4), (2, 2)])
def test_small_adjoints_beside_large_ones(dims, order, decades):
    """A plasma at rest without fields: lamE of a node is the sum of 2 hqm lamU
    times the weights, all positive, so that its error is at most that of one
    term and of the few additions of tiles' sums.  A weight is off by at most
    64 half-units as a polynomial and, with offsets that keep 0.1 away from the
    ends of every piece, 4 / 0.1 / 2 as its argument is rounded; the products,
    the constant and at most 20 tiles' or slabs' sums add 30.  The adjoints
    fall by `decades` per cell along x, 14 decades over a tile."""
    n = (24, 16, 12) if dims == 3 else (48, 32)
    w = I.Workload("adjn", dims, n, (0.2, 0.25, 0.2)[:dims], order, 4, 0.0, 1, seed=I.SEED_BASE + 180 + order)
    pl, E, B = inputs_for(w)
    rng = np.random.default_rng(12 + order)
    pl.off[:dims] = (0.1 + 0.3 * rng.random((dims, pl.np))).astype(np.float32)
    lam = (1.0 + rng.random((3, pl.np))) * 10.0 ** (-decades * ((pl.cell % n[0]) % 8))
    lam = lam.astype(np.float32).astype(np.float64)
    got, ref = _lam_e(w, 4, pl, E, B, lam), _lam_e(w, 8, pl, E, B, lam)
    assert np.abs(ref).min() > 0
    off = np.abs(got / ref - 1).max()
    tol = (84 * dims + 30) * 2.0 ** -24
    print("adjoint nodes", dims, order, decades, off, tol, flush=True)
    assert off <= tol
