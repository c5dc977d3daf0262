"""The occupied space at sizes on both sides of the purification's tile edges (16 up to N = 352, 32 up to N = 704, 48
beyond) and of single tiles: the density of a converged SCF is a projector with the right trace that commutes with F."""
import pytest

from tests.gpu_common import need_gpu, problem, torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,nc", [("tiny", 1), ("tiny", 4), ("tiny", 5), ("n400", 35), ("n400", 36), ("n400", 70),
                                     ("n400", 71)])
def test_projector(name, nc):
    need_gpu()
    import synth
    s = synth.config_system(name, n_centres=nc, seed=90 + nc)
    pr = problem(s)
    res, C, F, D = pr.energy()
    assert res["converged"]
    x = torch.tensor(s.xyz, device="cuda")[torch.tensor(s.fn_centre, device="cuda").long()]
    a = torch.tensor(s.fn_exp, device="cuda")
    p = a[:, None] + a[None]
    r2 = ((x[:, None] - x[None]) ** 2).sum(-1)
    S = (4 * a[:, None] * a[None]) ** 0.75 / p ** 1.5 * torch.exp(-a[:, None] * a[None] / p * r2)
    DS = D @ S
    # C is orthonormalised by two Cholesky QR passes: rounding of N-long sums
    assert float((DS @ D - 2 * D).abs().max()) < 1e-11 * float(D.abs().max())
    assert abs(float(torch.trace(DS)) - 2 * s.n_occ) < 1e-9
    assert float((F @ D @ S - S @ D @ F).abs().max()) < 1e-7
