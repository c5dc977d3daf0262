"""The pairs in another order than the list that build_3c writes: the columns of the fitted tensor permuted with them.
J, K, gamma and the gradient are sums over the pairs, so only their rounding may change."""
import numpy as np
import pytest

from tests.gpu_common import dev, need_gpu, problem, torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nc", [3, 17, 37])
def test_permuted_pairs(nc):
    need_gpu()
    import synth
    s = synth.config_system("n400", n_centres=nc, seed=9)
    pr = problem(s)
    C, F = dev(synth.random_coeffs(s.N, s.n_occ, 1)), dev(synth.random_coeffs(s.N, s.N, 2))
    F = F + F.T

    def results():
        J, K, g = pr.fock_jk(C)
        Jd, Kd = pr.fock_jk_density(2.0 * C @ C.T)
        return [x.clone() for x in (J, K, g, Jd, Kd, pr.gradient(C, F))]

    ref = results()
    order = torch.as_tensor(np.random.default_rng(nc).permutation(pr.n_pairs), device="cuda")
    pr.pairs, pr.T = pr.pairs[order].contiguous(), pr.T[:, order].contiguous()
    for a, b in zip(ref, results()):
        # sums of at most N_aux * N * n_occ products in another order; the gradient's terms cancel, 1e3 over its largest
        assert float((a - b).abs().max()) < 1e-10 * max(float(a.abs().max()), 1.0)
