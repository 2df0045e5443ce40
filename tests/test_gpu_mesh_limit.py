"""Diagnostics of a mesh near the largest number of cells (2^31 - 2)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_diagnostics_of_the_largest_meshes():
    """The sums over cells run to 2^31 - 42k cells without a cell index leaving
    its range: with every sample of E and B one, the field energy is a whole
    number of half cells (exact: its sums are integers below 2^53)."""
    from paper_1310_0930_amd import pic as P
    n = (46340, 46341)
    ncell = n[0] * n[1]
    assert 2 ** 31 - 2 ** 19 < ncell < 2 ** 31 - 1
    ctx = P.pic_create(P.make_config(2, n, (1.0, 1.0), 0.5, 1, real_bytes=4))
    try:
        ones = torch.ones(ncell, dtype=torch.float32, device="cuda")
        rho = torch.empty(ncell, dtype=torch.float64, device="cuda")
        ws = torch.zeros(P.pic_workspace_bytes(ctx, 0), dtype=torch.uint8, device="cuda")
        none = torch.zeros((3, 1), device="cuda")
        parts = P.particles_struct(0, torch.zeros(1, dtype=torch.int32, device="cuda"), none, none)
        F = [ones] * 3
        d = P.pic_diagnostics(ctx, parts, P.fields_struct(F, F, F), None, None, rho.data_ptr(), None,
                              ws.data_ptr()).as_dict()
        assert d["w_field"] == 3.0 * ncell
        assert d["rho_max"] == 0.0 and d["gauss_max"] == 0.0 and d["n_alive"] == 0
    finally:
        P.pic_destroy(ctx)
