"""Patches with Neumann slots by several fine steps per launch against single
steps and their perimeter kernel: every node takes the same operations, so FP64
and FP32 states and counts are equal bit for bit; FP16 shifted storage rounds to
binary16 once per launch instead of once per step (4e-3 of the largest value, the
bound of the other multi-step tests).  The closed-form closure itself is held to
the oracle's Newton iteration."""
import numpy as np
import pytest

from paper_1601_02708_amd import inputs

pytestmark = pytest.mark.gpu


def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1601_02708_amd import hyb
    return hyb


def _handle(hyb, N, eta, precision, rng):
    solid = np.zeros((N, N), np.uint8)
    if N > 60:
        j, i = np.mgrid[0:N, 0:N]
        solid = (((i + j // 7) % 37 - 18) ** 2 + ((j + i // 11) % 41 - 20) ** 2 <= 120).astype(np.uint8)
        solid[:3], solid[-3:], solid[:, :3], solid[:, -3:] = 0, 0, 0, 0
    v = rng.uniform(-0.05, 0.05, (2, N, N)).astype(np.float32) * (solid == 0)
    kind = rng.integers(0, 2, 4 * (N - 1)).astype(np.int8)       # corners and edges of both kinds
    a, b = rng.uniform(0.2, 0.6, (2, 4 * (N - 1)))
    # outward fluxes small enough to be met, and some that are not (R' <= 0)
    a[kind == 1], b[kind == 1] = rng.uniform(-0.02, 0.02, (2, int(kind.sum())))
    f0 = inputs.random_populations(N, 7, lo=0.03, hi=0.06)
    f0[:, solid != 0] = 0.0
    g = hyb.Hybrid(N=N, x0=0, y0=0, u0=np.full((N, N), 0.4), vx=v[0], vy=v[1], D=0.02, eta=eta, precision=precision,
                   solid=solid, k=1e-3)
    if precision != "fp16s":
        g.set_populations(f0)
    g.set_boundary(a, b, kind)
    return g, (solid, v, kind, a, b, f0)


# 9: one tile, all perimeter; 65: a last tile of one column; 1409: strips inside the frame
@pytest.mark.parametrize("N,spl,eta", [(9, 2, 4), (9, 5, 5), (65, 3, 6), (65, 4, 9), (200, 2, 5), (200, 5, 7),
                                       (1409, 4, 5), (1409, 5, 5)])
@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16s"])
def test_outlet_launches_equal_single_steps(precision, N, spl, eta):
    hyb = _gpu()
    out = []
    for s in (spl, 1):
        g, _ = _handle(hyb, N, eta, precision, np.random.default_rng(N + eta))
        g.set_steps_per_launch(s)
        g.lbm_substeps(eta, restart=1)
        g.commit()
        st = g.stats()
        out.append((g.get_populations(), st["infeasible"], st["nonfinite"]))
        g.close()
    if precision == "fp16s":
        assert np.abs(out[0][0] - out[1][0]).max() <= 4e-3 * np.abs(out[1][0]).max()
    else:
        assert np.array_equal(out[0][0], out[1][0]) and out[0][1:] == out[1][1:]


def test_closed_form_closure_matches_newton(orc):
    hyb = _gpu()
    N, eta = 21, 3
    g, (solid, v, kind, a, b, f0) = _handle(hyb, N, eta, "fp64", np.random.default_rng(5))
    g.lbm_substeps(eta, restart=1)
    g.commit()
    lat = orc.Lattice(N, 0.02 * 3 + 0.5, v[0].astype(np.float64), v[1].astype(np.float64), solid=solid, k=1e-3,
                      bc_kind=kind)
    f, bad = f0.copy(), 0
    for t in range(1, eta + 1):
        f, n = lat.substep(f, (1 - t / eta) * a + t / eta * b)
        bad += n
    # Newton stops at steps of 4 eps (1 + |g|), |g| < 4: 5e-15 of values below 0.2, over three steps
    assert np.abs(g.get_populations() - f).max() <= 1e-14 and g.stats()["infeasible"] == bad
    g.close()
