"""hyb_query's workspace holds what hyb_create lays out: a descriptor that does
not name eta yet gets room for every eta (no GPU needed)."""
import ctypes

import pytest


@pytest.mark.parametrize("N", [150, 170, 180, 188, 192, 196, 1000])
@pytest.mark.parametrize("precision", [0, 1, 2])
def test_query_without_eta_covers_every_eta(N, precision):
    from paper_1601_02708_amd import hyb
    lib = hyb.load()
    mesh = hyb.HybMesh(16, 4094.0, 0.0, 1, 1, None)

    def query(eta):
        lat = hyb.HybLattice()
        lat.N, lat.precision, lat.eta = N, precision, eta
        fb, wb = ctypes.c_size_t(), ctypes.c_size_t()
        assert lib.hyb_query(ctypes.addressof(mesh), ctypes.addressof(lat), ctypes.addressof(fb),
                             ctypes.addressof(wb)) == hyb.HYB_OK
        return wb.value

    assert query(0) >= max(query(eta) for eta in list(range(1, 60)) + [10 ** 9])
