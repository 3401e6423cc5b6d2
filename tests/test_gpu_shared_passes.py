"""hyb_step, whose later Schwarz passes sweep only the frame that their interface
values reach, against the same step through the separate calls, whose passes
all sweep the whole patch: the shared nodes take the same operations from the
same state, so states, coarse solution and counts are equal bit for bit."""
import numpy as np
import pytest

from paper_1601_02708_amd import configs

pytestmark = pytest.mark.gpu


def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1601_02708_amd import hyb
    return hyb


def _separate(hyb, g, passes):
    for _ in range(passes):
        g.interface_exchange(hyb.HYB_F2C)
        g.coarse_step(200)
        g.interface_exchange(hyb.HYB_C2F)
        g.lbm_substeps(g.eta, restart=1)
    g.commit()


# no whole tile inside the frame (N = 100); the smallest hole (N = 201); holes
# of one and two launches, ragged right and top tiles, three passes, overlap
@pytest.mark.parametrize("precision,N,eta,spl,passes,overlap",
                         [("fp64", 100, 4, 4, 2, 0), ("fp64", 201, 4, 4, 2, 1), ("fp64", 261, 7, 4, 3, 2),
                          ("fp32", 330, 10, 5, 2, 0), ("fp32", 395, 10, 5, 3, 2), ("fp32", 257, 2, 5, 2, 1),
                          ("fp32", 257, 9, 3, 2, 1), ("fp16s", 395, 8, 4, 2, 2), ("fp16s", 260, 5, 5, 3, 0),
                          ("fp64", 1473, 7, 4, 2, 1),
                          # three launches (4 + 3 + 3, 4 + 4 + 4), four and six (the fourth state), five without it
                          ("fp64", 395, 10, 4, 3, 0), ("fp16s", 330, 12, 4, 2, 1), ("fp32", 458, 15, 5, 2, 2),
                          ("fp64", 395, 13, 4, 3, 0), ("fp32", 523, 20, 5, 3, 1), ("fp32", 600, 26, 5, 2, 0),
                          ("fp32", 330, 10, 2, 2, 0)])
def test_shared_passes_equal_whole_passes(precision, N, eta, spl, passes, overlap):
    hyb = _gpu()
    p = configs.build_problem(configs.PORE2048.replace(N=N, M=16, eta=eta, porosity=0.8 if N < 1000 else None))
    out = []
    for whole in (False, True):
        g = hyb.Hybrid.from_problem(p, precision=precision)
        g.set_steps_per_launch(spl)
        g.set_overlap(overlap)
        for _ in range(3):
            _separate(hyb, g, passes) if whole else g.step(passes)
        s = g.stats()
        out.append((g.get_populations(), g.concentration(hyb.HYB_COARSE), s["infeasible"], s["fine_steps"]))
        g.close()
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
    assert out[0][2:] == out[1][2:]


@pytest.mark.parametrize("eta,passes", [(4, 2), (10, 3), (15, 2), (20, 3)])
def test_nonfinite_nodes_of_shared_passes_are_counted_in_every_pass(eta, passes):
    """A NaN far from the perimeter: the step fails as the separate calls do,
    with the same count and the same state left behind."""
    hyb = _gpu()
    p = configs.build_problem(configs.PORE2048.replace(N=395, M=16, eta=eta, porosity=None))
    out = []
    for whole in (False, True):
        g = hyb.Hybrid.from_problem(p, precision="fp32")
        f = g.get_populations()
        f[3, 200, 190] = np.nan
        g.set_populations(f)
        with pytest.raises(hyb.HybError) as e:
            _separate(hyb, g, passes) if whole else g.step(passes)
        assert e.value.code == hyb.HYB_ENONFINITE
        s = g.stats()
        out.append((g.get_populations(), s["nonfinite"], s["infeasible"]))
        g.close()
    assert np.array_equal(out[0][0], out[1][0], equal_nan=True)
    assert out[0][1:] == out[1][1:] and out[0][1] > 0


# launches of two to five steps, two to four a pass; the solids around the hole
# dissolve away within the run
@pytest.mark.parametrize("precision,N,eta,passes", [("fp64", 201, 5, 2), ("fp64", 330, 10, 3), ("fp32", 523, 20, 2),
                                                    ("fp32", 330, 8, 2), ("fp16s", 330, 13, 2)])
def test_shared_passes_of_dissolving_solids(precision, N, eta, passes):
    """The masses too: a later pass sums the link fluxes of the frame anew and
    keeps those of the shared nodes."""
    hyb = _gpu()
    p = configs.build_problem(configs.PORE2048.replace(N=N, M=16, eta=eta, porosity=0.7))
    mass = np.random.default_rng(8).uniform(0.002, 0.01, (N, N))
    out = []
    for whole in (False, True):
        g = hyb.Hybrid.from_problem(p, precision=precision, dissolution=True)
        g.set_dissolution(0.2, 1.0, mass)
        for _ in range(3):
            _separate(hyb, g, passes) if whole else g.step(passes)
        out.append((g.get_populations(), g.concentration(hyb.HYB_COARSE)) + tuple(g.dissolution_state()[:2]))
        conv = g.dissolution_state()[2]
        g.close()
    assert conv > 0
    for x, y in zip(*out):
        assert np.array_equal(x, y)
