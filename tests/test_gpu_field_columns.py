"""The field advance by columns of four planes where four divides the planes
(no column is short): against the oracle, as for the other grids."""
import pytest

from test_gpu_fields import test_field_advance_against_the_oracle as _check

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rb", [8, 4])
@pytest.mark.parametrize("n,bc", [((96, 80, 72), (0, 0, 0)), ((67, 4, 1960), (0, 0, 0)),
                                  ((96, 80, 72), (1, 1, 1))])
def test_whole_columns(n, bc, rb):
    _check(n, bc, rb)
