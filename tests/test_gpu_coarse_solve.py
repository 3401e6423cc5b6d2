"""The one-launch coarse solve (tiles of 17 x 17 mesh nodes, up to 64 of them)
against the oracle's banded LU, at the meshes where its tiling can go wrong: one
tile exactly (M = 16), a last tile one node wide (17), two (18, 35), a ragged
one, the most tiles (135), and the first mesh that the per-product kernels take
(136).  The same residual bound as before (1e-14 of the right-hand side) on
operators of condition number of a few tens: 1e-12."""
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


@pytest.mark.parametrize("M,N", [(8, 64), (16, 64), (17, 64), (18, 64), (35, 101), (50, 101), (135, 160), (136, 160)])
def test_solve_matches_direct(orc, M, N):
    hyb, _ = _gpu()
    p = configs.build_problem(configs.SMALL.replace(N=N, M=M, k=1e-3))
    g = hyb.Hybrid.from_problem(p)
    o = orc.HybridOracle(p)
    for _ in range(2):
        g.step(p.cfg.max_iter)
        s = g.stats()
        assert s["krylov_converged"] == 1 and s["krylov_relres"] <= 1e-14 and 0 < s["krylov_iters"] < 40
    o.run(2)
    assert _rel(g.concentration(hyb.HYB_COARSE), o.d) <= 1e-12
    assert _rel(g.concentration(), o.fine_concentration()) <= 1e-12
    g.close()


@pytest.mark.parametrize("M,N", [(16, 64), (17, 64), (50, 101), (136, 160)])
def test_transposed_solve_matches_direct(orc, M, N):
    from oracle.hybrid_adjoint import HybridStepAdjoint
    hyb, torch = _gpu()
    p = configs.build_problem(configs.SMALL.replace(N=N, M=M, k=1e-3))
    g = hyb.Hybrid.from_problem(p)
    rng = np.random.default_rng(M)
    lam_f, lam_d = rng.standard_normal((9, N, N)), rng.standard_normal((M + 1) ** 2)
    lf, ld = torch.from_numpy(lam_f).to(g.dev), torch.from_numpy(lam_d).to(g.dev)
    of, od = torch.empty_like(lf), torch.empty_like(ld)
    tape = g.step_tape(2)
    F0, d0 = g.get_populations(), g.concentration(hyb.HYB_COARSE).reshape(-1)
    g.step_record(2, tape)
    g.step_adjoint(tape, lf, ld, of, od)
    adj = HybridStepAdjoint(orc.HybridOracle(p))
    _, _, otape = adj.forward(F0, d0)
    rf, rd, _ = adj.adjoint(otape, lam_f, lam_d)
    assert _rel(of.cpu().numpy(), rf) <= 1e-11 and _rel(od.cpu().numpy(), rd) <= 1e-11
    g.close()


def test_two_handles_solve_on_two_streams():
    """Solves of two handles in flight together on two streams give each
    handle's own result (their words lie in their own workspaces)."""
    hyb, torch = _gpu()
    ps = [configs.build_problem(configs.SMALL.replace(N=101, M=M, k=1e-3, seed=M)) for M in (50, 67)]
    want = []
    for p in ps:
        g = hyb.Hybrid.from_problem(p)
        for _ in range(4):
            g.step(2)
        want.append(g.concentration(hyb.HYB_COARSE))
        g.close()
    hs = []
    for p in ps:
        with torch.cuda.stream(torch.cuda.Stream()):
            hs.append(hyb.Hybrid.from_problem(p))
    torch.cuda.synchronize()
    for _ in range(4):
        for g in hs:
            for _ in range(2):
                g.interface_exchange(hyb.HYB_F2C)
                g.coarse_step(200)
                g.interface_exchange(hyb.HYB_C2F)
                g.lbm_substeps(g.eta, restart=1)
        for g in hs:
            g.commit()
    for g, w in zip(hs, want):
        assert np.array_equal(g.concentration(hyb.HYB_COARSE), w)
        g.close()
