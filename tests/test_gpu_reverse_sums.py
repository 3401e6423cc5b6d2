"""What the Schwarz passes of a coarse step add to dJ/df* and dJ/dk is added in
FP64, whatever the storage type: a pass's part keeps its digits beside a cotangent
that is ten million times larger.

lam_f is 1 far from the perimeter and 0 elsewhere, so it reaches no interface value
and the last pass alone carries it; lam_d reaches the earlier passes through the
coarse step.  The reverse mode is linear and every pass is swept apart, so the
result with both less that with lam_f alone is that with lam_d alone, to the FP64
roundings of a sum per pass and one for the transfer (of the larger part)."""
import numpy as np
import pytest

from paper_1601_02708_amd import configs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,passes,eta", [(200, 2, 4), (1450, 2, 5), (1450, 3, 4)])
def test_passes_are_added_in_fp64(N, passes, eta):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1601_02708_amd import hyb
    M = 64 if N > 1000 else 24
    p = configs.build_problem(configs.PORE2048.replace(N=N, M=M, eta=eta, max_iter=passes, k=1e-4))
    g = hyb.Hybrid.from_problem(p, precision="fp32")
    tape = g.step_tape(passes)
    g.step_record(passes, tape)
    d = 3 * eta
    lam_f = torch.zeros((9, N, N), dtype=torch.float64, device=g.dev)
    lam_f[:, d:-d, d:-d] = 1.0
    lam_f *= torch.from_numpy((p.solid == 0) * 1.0).to(g.dev)
    lam_d = 1e-6 * torch.from_numpy(np.random.default_rng(3).standard_normal((M + 1) ** 2)).to(g.dev)

    def reverse(f, dd):
        out, out_d = torch.full_like(f, float("nan")), torch.empty_like(lam_d)
        gk = torch.zeros((N, N), dtype=torch.float64, device=g.dev)
        g.step_adjoint(tape, f, dd, out, out_d, gk)
        return out, gk

    both, large, small = reverse(lam_f, lam_d), reverse(lam_f, torch.zeros_like(lam_d)), reverse(0 * lam_f, lam_d)
    for x, y, z in zip(both, large, small):
        inner = z[..., d:-d, d:-d].abs().max()
        assert 0 < inner < 1e-5 * y.abs().max()
        off = (x - y - z).abs().max()
        assert off <= 2 * (2 * passes + 2) * 2.0 ** -53 * y.abs().max(), (float(off), float(inner))
    g.close()
