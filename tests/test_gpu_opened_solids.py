"""Sweeps leave what is stored at the solid nodes of a handle whose solids can
change: a node that hyb_set_solids opens starts from zeros, on small patches
(tiles) and on large ones, whose inner nodes go to strips where solids stay."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [200, 1450])
@pytest.mark.parametrize("precision,record", [("fp64", False), ("fp32", False), ("fp32", True)])
def test_opened_nodes_hold_zeros(N, precision, record):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1601_02708_amd import hyb
    j, i = np.mgrid[0:N, 0:N]
    solid = (((i % 50) - 25) ** 2 + ((j % 50) - 25) ** 2 <= 120) & (i > 3) & (j > 3) & (i < N - 4) & (j < N - 4)
    v = np.full((N, N), 0.03, np.float32) * ~solid
    g = hyb.Hybrid(N=N, x0=0, y0=0, u0=np.full((N, N), 0.4), vx=v, vy=0 * v, D=0.02, eta=4, precision=precision,
                   solid=solid.astype(np.uint8), dissolution=True)
    g.set_boundary(np.full(4 * (N - 1), 0.5), np.full(4 * (N - 1), 0.6))
    if record:
        g.substeps_record(4, g.adjoint_tape(4))
    else:
        g.lbm_substeps(4, restart=1)
    g.commit()
    left = solid & (i % 100 < 50)
    g.set_solids(left.astype(np.uint8), np.where(left, 1.0, 0.0))
    u = g.concentration()
    assert (u[solid & ~left] == 0).all() and (u[~solid] > 0.3).all()
    g.close()
