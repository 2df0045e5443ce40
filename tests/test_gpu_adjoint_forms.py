"""The step adjoint's LDS forms against global memory, element by element, where
the launch's rules choose another form: meshes of many tiles per CU (2D
workgroups of 4 wavefronts; 3D in two phases from quadratic order on) and of
few, open faces, ragged last tiles, cubic FP64."""
import pytest

from paper_1310_0930_amd import inputs as I
from test_gpu_adjoint import _tiled_vs_global

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rb", [4, 8])
@pytest.mark.parametrize("order", [1, 2, 3, 4])
def test_many_tiles_2d(order, rb):
    """25 x 22 tiles."""
    w = I.Workload("adjf2", 2, (400, 341), (0.1, 0.2), order, 2, 0.2, 1, bc=(0, 1), ramp_cells=6.0,
                   seed=I.SEED_BASE + 220 + order)
    _tiled_vs_global(w, rb, 51 + order)


@pytest.mark.parametrize("rb", [4, 8])
@pytest.mark.parametrize("order", [1, 2, 3, 4])
def test_many_tiles_3d(order, rb):
    """6 x 6 x 8 tiles of 8^3 cells (more of them where tiles are smaller)."""
    w = I.Workload("adjf3", 3, (44, 41, 58), (0.2, 0.25, 0.2), order, 1, 0.3, 1, bc=(0, 1, 1),
                   ramp_cells=4.0, seed=I.SEED_BASE + 230 + order)
    _tiled_vs_global(w, rb, 61 + order)


@pytest.mark.parametrize("bc", [(0, 1, 0), (0, 1, 1), (1, 1, 1)])
@pytest.mark.parametrize("n", [(24, 16, 20), (12, 10, 9)])
def test_cubic_fp64(n, bc):
    w = I.Workload("adjf33", 3, n, (0.2, 0.25, 0.2), 3, 4, 0.3, 1, bc=bc, ramp_cells=4.0,
                   seed=I.SEED_BASE + 240 + sum(bc))
    _tiled_vs_global(w, 8, 71 + sum(bc))
