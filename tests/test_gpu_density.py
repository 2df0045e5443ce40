"""The tile pass of the charge density against the global-memory pass, from one
particle per cell to all of them on one node."""
import numpy as np
import pytest

from paper_1310_0930_amd import inputs as I

from _parity import gpu_sim, inputs_for

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _both(w, rb, pl, E, B):
    from paper_1310_0930_amd import pic as P
    sim = gpu_sim(w, rb, pl, E, B)
    sim.sort()
    out = []
    for ws in (sim.ws.data_ptr(), None):
        rho = torch.empty(sim.ncell, dtype=torch.float64, device=sim.device)
        P.pic_deposit_rho(sim.ctx, sim._parts, rho.data_ptr(), ws)
        out.append(rho.cpu().numpy())
    return out


@pytest.mark.parametrize("rb", [4, 8])
@pytest.mark.parametrize("dims,order,ppc,crowded", [
    (3, 1, 4, False), (3, 2, 1, False), (3, 2, 2, False), (3, 2, 20, False), (3, 3, 9, False),
    (3, 4, 4, False), (2, 2, 4, False), (2, 3, 2, False), (2, 4, 20, False), (3, 2, 9, True),
    (3, 3, 9, True), (3, 4, 9, True), (2, 2, 9, True), (2, 3, 9, True), (2, 4, 9, True)])
def test_density_of_a_tile_equals_global_memory(dims, order, ppc, crowded, rb):
    """Sums of m <= (order + 1)^dims ppc weights (crowded: every particle on the
    one node of the largest weight, which takes the integer sums to their bound):
    in double each is rounded m times, a weight in fixed point to half of 2^-52
    at the coarsest for up to 4096 particles in a tile, 4 times that here."""
    n = (21, 16, 12) if dims == 3 else (40, 36)
    w = I.Workload("w_rho", dims, n, (0.2,) * dims, order, ppc, 0.1, 1, bc=(0, 1, 0)[:dims],
                   seed=I.SEED_BASE + 191 + order)
    pl, E, B = inputs_for(w)
    m = (order + 1) ** dims * ppc
    if crowded:
        pl = I.Plasma(np.full_like(pl.cell, pl.cell[pl.np // 2]),
                      np.full_like(pl.off, 0.0), pl.u, None, pl.q_const)
        m = pl.np
    tiled, glob = _both(w, rb, pl, E, B)
    scale = np.abs(glob).max()
    assert scale > 0
    q = abs(w.q_const)
    assert np.abs(tiled - glob).max() <= 2.0 ** -53 * m * scale + 2.0 ** -51 * m * q
