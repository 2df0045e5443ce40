"""The tile sort of particles in no order, over more tiles than a workgroup's
tile table holds and on chunks that end at or beside a multiple of its sizes."""
import numpy as np
import pytest

from paper_1310_0930_amd import inputs as I
from _parity import gpu_sim, inputs_for
from test_gpu_parity import _check_sorted

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SHAPES = [  # 16 x 20 and 5 x 5 x 17 tiles, and one tile
    ((256, 320), 2), ((40, 36, 130), 2), ((7, 5), 2)]


@pytest.mark.parametrize("rb", [8, 4])
@pytest.mark.parametrize("n,order", SHAPES)
@pytest.mark.parametrize("keep", [0, 1, 1023, 1025, 4096, 4097, None])
def test_sort_of_shuffled_particles_over_many_tiles(n, order, rb, keep):
    """Counts, order and payload are whole numbers or copied bits: exact."""
    dims = len(n)
    w = I.Workload("w_sort_many", dims, n, (0.2,) * dims, order, 2, 0.3, 1, seed=I.SEED_BASE + 131 + dims)
    pl, E, B = inputs_for(w)
    rng = np.random.default_rng(6)
    perm = rng.permutation(pl.np)[:keep]
    pl = I.Plasma(pl.cell[perm].copy(), pl.off[:, perm].copy(), pl.u[:, perm].copy(), None, pl.q_const)
    pl.cell[rng.random(pl.np) < 0.02] = -1
    sim = gpu_sim(w, rb, pl, E, B)
    sim.sort()
    assert sim.np == int(np.sum(pl.cell >= 0))
    _check_sorted(w, rb, pl, sim.download())
