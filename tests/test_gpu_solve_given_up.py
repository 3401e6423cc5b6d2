"""The one-launch coarse solve where its workgroups give up waiting for each other
(hyb_set_solve_polls(0): each at its first wait, so that every kernel ends at
once) and one of them solves alone, against the same calls that wait.  Both stop
at 1e-14 of the right-hand side, on operators of condition number of a few tens:
1e-12, and 1e-11 for the transposed solves, whose right-hand side is a product."""
import numpy as np
import pytest

from paper_1601_02708_amd import configs

pytestmark = pytest.mark.gpu


def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1601_02708_amd import hyb
    return hyb, torch


def _rel(a, b):
    a, b = np.asarray(a, float).ravel(), np.asarray(b, float).ravel()
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def _by_hand(hyb, g, passes):
    for _ in range(passes):
        g.interface_exchange(hyb.HYB_F2C)
        g.coarse_step(200)
        g.interface_exchange(hyb.HYB_C2F)
        g.lbm_substeps(g.eta, restart=1)
    g.commit()


@pytest.mark.parametrize("M,N", [(17, 64), (50, 101), (135, 160)])
@pytest.mark.parametrize("by_hand", [False, True])
def test_step_goes_on(M, N, by_hand):
    hyb, _ = _gpu()
    p = configs.build_problem(configs.SMALL.replace(N=N, M=M, k=1e-3))
    got = []
    for polls in (-1, 0):
        g = hyb.Hybrid.from_problem(p)
        g.set_solve_polls(polls)
        for step in range(3):           # (after the first the handle takes a launch per product)
            if by_hand:
                _by_hand(hyb, g, p.cfg.max_iter)
            else:
                g.step(p.cfg.max_iter)
            s = g.stats()
            assert s["krylov_converged"] == 1 and s["krylov_relres"] <= 1e-14
            if step == 1:
                g.set_solve_polls(polls)
        got.append([g.concentration(hyb.HYB_COARSE), g.concentration()])
        g.close()
    for x, y in zip(*got):
        assert _rel(x, y) <= 1e-12


def test_group_goes_on():
    hyb, _ = _gpu()
    mp = configs.build_multi(65, 40, 260.0, [(30.0, 80.0), (150.0, 80.0)], D=1e-2, k=1e-3, eta=5, max_iter=2)
    got = []
    for polls in (-1, 0):
        ps = [hyb.Hybrid(N=p.N, x0=p.x0, y0=p.y0, u0=p.u0_fine, vx=p.vx, vy=p.vy, D=mp.D, eta=mp.eta, solid=p.solid,
                         k=mp.k) for p in mp.patches]
        g = hyb.HybridGroup(ps, dict(M=mp.M, L=mp.L, outer_value=0.0, overlap_elems=mp.overlap_elems, supg=mp.supg,
                                     d0=mp.u0_coarse, v=mp.vc), mp.D, mp.k)
        g.set_solve_polls(polls)
        for _ in range(2):
            g.step(2)
        got.append([g.coarse()] + [p.concentration() for p in ps])
        g.close()
    for x, y in zip(*got):
        assert _rel(x, y) <= 1e-12


@pytest.mark.parametrize("M,N", [(17, 64), (50, 101)])
def test_reverse_mode_goes_on(M, N):
    """No error, and each gradient added to once."""
    hyb, torch = _gpu()
    p = configs.build_problem(configs.SMALL.replace(N=N, M=M, k=1e-3))
    rng = np.random.default_rng(M)
    lam_f, lam_d = rng.standard_normal((9, N, N)), rng.standard_normal((M + 1) ** 2)
    got = []
    for polls in (-1, 0):
        g = hyb.Hybrid.from_problem(p)
        lf, ld = torch.from_numpy(lam_f).to(g.dev), torch.from_numpy(lam_d).to(g.dev)
        of, od = torch.empty_like(lf), torch.empty_like(ld)
        gk, go = torch.ones((N, N), dtype=torch.float64, device=g.dev), torch.ones_like(ld)
        tape = g.step_tape(2)
        g.step_record(2, tape)
        g.set_solve_polls(polls)
        g.step_adjoint(tape, lf, ld, of, od, gk, go)
        got.append([x.cpu().numpy() for x in (of, od, gk, go)])
        g.close()
    for x, y in zip(*got):
        assert _rel(x, y) <= 1e-11


def test_solve_beside_strips():
    """36 workgroups that wait for each other while strips of the next fine steps
    fill the chip and its memory, every overlap depth."""
    hyb, _ = _gpu()
    N, M = 1500, 100
    p = configs.build_problem(configs.PORE2048.replace(N=N, M=M, k=1e-4))
    got = []
    for polls, depth in ((0, 0), (-1, 0), (-1, 1), (-1, 2)):
        g = hyb.Hybrid.from_problem(p, precision="fp64")
        g.set_solve_polls(polls)
        g.set_overlap(depth)
        for _ in range(4):
            g.step(2)
        got.append([g.concentration(hyb.HYB_COARSE), g.concentration()])
        g.close()
    for run in got[1:]:
        assert _rel(run[0], got[0][0]) <= 1e-12 and _rel(run[1], got[0][1]) <= 1e-12
    assert all(np.array_equal(x, y) for run in got[2:] for x, y in zip(run, got[1]))
