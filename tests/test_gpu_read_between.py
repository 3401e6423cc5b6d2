"""Reading the state between hyb_step_record and hyb_step_adjoint (which the
handle allows: nothing changes) leaves the gradients as they are, bit for bit."""
import numpy as np
import pytest

from paper_1601_02708_amd import configs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dissolution", [False, True])
@pytest.mark.parametrize("passes,M", [(1, 24), (2, 96)])         # (96: elements shorter than the fine steps reach)
def test_readouts_between_record_and_adjoint(dissolution, passes, M):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1601_02708_amd import hyb
    p = configs.build_problem(configs.PORE2048.replace(N=193, M=M, eta=5, k=1e-3))
    N = p.cfg.N
    g = hyb.Hybrid.from_problem(p, precision="fp64", dissolution=dissolution)
    if dissolution:
        g.set_dissolution(0.1, 1.0, np.full((N, N), 0.05))
    tape = g.step_tape(passes)
    rng = np.random.default_rng(0)
    lam_f = torch.from_numpy(rng.standard_normal((9, N, N))).to(g.dev)
    lam_d = torch.from_numpy(rng.standard_normal((M + 1) ** 2)).to(g.dev)

    def reverse():
        out_f, out_d = torch.empty_like(lam_f), torch.empty_like(lam_d)
        gk = torch.zeros((N, N), dtype=torch.float64, device=g.dev)
        g.step_adjoint(tape, lam_f, lam_d, out_f, out_d, gk)
        return [x.cpu().numpy() for x in (out_f, out_d, gk)]

    for _ in range(3):                  # every buffer takes its turn as the step's start
        g.step_record(passes, tape)
        want = reverse()
        g.concentration()
        g.get_populations()
        g.stats()
        for x, y in zip(reverse(), want):
            assert np.array_equal(x, y)
    g.close()
