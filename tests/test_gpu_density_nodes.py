"""The charge density node by node, also where a node holds a small charge (the
edge of a plasma, a thin plasma beside a dense one): against sums in extended
precision."""
import numpy as np
import pytest

from paper_1310_0930_amd import inputs as I

from _parity import gpu_sim, inputs_for

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _weights(order, o):
    """B-spline weights of the nodes first .. first + order, and first."""
    L = np.longdouble
    k = np.zeros(o.shape, np.int64) if order & 1 else (o >= 0.5).astype(np.int64)
    x = o - k
    if order == 1:
        w = [1 - x, x]
    elif order == 2:
        w = [(L(0.5) - x) ** 2 / 2, L(0.75) - x * x, (L(0.5) + x) ** 2 / 2]
    elif order == 3:
        w = [(1 - x) ** 3 / 6, (4 - 6 * x ** 2 + 3 * x ** 3) / 6,
             (1 + 3 * x + 3 * x ** 2 - 3 * x ** 3) / 6, x ** 3 / 6]
    else:
        w = [(1 - 2 * x) ** 4 / 384, (19 + x * (-44 + x * (24 + x * (16 - 16 * x)))) / 96,
             (115 + x * x * (-120 + 48 * x * x)) / 192,
             (19 + x * (44 + x * (24 + x * (-16 - 16 * x)))) / 96, (1 + 2 * x) ** 4 / 384]
    return w, k - order // 2


def _exact(w, cell, off, q):
    n = w.n3
    c = cell.astype(np.int64)
    at = [c % n[0], c // n[0] % n[1], c // (n[0] * n[1])]
    per = [_weights(w.order, off[d].astype(np.longdouble)) for d in range(w.dims)]
    rho = np.zeros(n[0] * n[1] * n[2], np.longdouble)
    for idx in np.ndindex(*(w.order + 1,) * w.dims):
        v, to = np.longdouble(q), 0
        for d in reversed(range(w.dims)):
            v = v * per[d][0][idx[d]]
            to = to * n[d] + (at[d] + per[d][1] + idx[d]) % n[d]
        np.add.at(rho, to, v)
    return rho


@pytest.mark.parametrize("rb", [4, 8])
@pytest.mark.parametrize("dims,order,ppc", [(3, 1, 8), (3, 2, 8), (3, 3, 8), (3, 4, 4), (3, 4, 2),
                                            (2, 2, 16), (2, 3, 9), (2, 4, 16)])
def test_density_of_every_node(dims, order, ppc, rb):
    """Half of the box is full, a quarter holds one particle in eight.  A node's
    sum is of at most m = (order + 1)^dims ppc terms of one sign, each rounded
    once as it is added; a term is a product of dims weights and the charge,
    and a weight is off by at most 64 half-units (the quartic's middle pieces
    cancel to a fifth of their terms; the others by 10 or less)."""
    n = (21, 16, 12) if dims == 3 else (56, 36)
    w = I.Workload("w_rho_nodes", dims, n, (0.2,) * dims, order, ppc, 0.1, 1,
                   seed=I.SEED_BASE + 211 + order)
    pl, E, B = inputs_for(w)
    x = pl.cell % n[0]
    some = np.random.default_rng(4).random(pl.np) < 0.125
    keep = (x < n[0] // 2) | ((x < 3 * n[0] // 4) & some)
    pl = I.Plasma(pl.cell[keep].copy(), pl.off[:, keep].copy(), pl.u[:, keep].copy(), None, pl.q_const)
    sim = gpu_sim(w, rb, pl, E, B)
    ref = _exact(w, pl.cell, pl.off, w.q_const)
    sim.sort()
    rho = sim.rho().cpu().numpy()
    tol = ((order + 1) ** dims * ppc + 64 * dims + 4) * 2.0 ** -53
    off = np.abs(rho - ref) / np.where(ref == 0, 1, np.abs(ref))
    print("density nodes", dims, order, ppc, rb, float(off.max()), tol, flush=True)
    assert off.max() <= tol
