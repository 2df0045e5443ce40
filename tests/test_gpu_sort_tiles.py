"""The tile sort on meshes of more tiles than one workgroup's share of the scan
(8192): exact, as for the smaller meshes."""
import pytest

from test_gpu_sort import test_sort_of_shuffled_particles_over_many_tiles as _check

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rb", [8, 4])
@pytest.mark.parametrize("n", [(2048, 2080), (1440, 1456), (168, 160, 176)])
def test_sort_over_more_tiles_than_a_chunk(n, rb):
    """16640 and 8190 tiles (three chunks and, with the dead bin, the last one
    full but for one count), 9240 tiles in 3D."""
    _check(n, 2, rb, 30001)
