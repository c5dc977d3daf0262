"""J and K of a density at sizes around the slabs, blocks and tiles of its kernels, against plain torch in FP64 from
the same fitted tensor; D with an antisymmetric part, which is not used."""
import numpy as np
import pytest

from tests.gpu_common import dev, need_gpu, problem, torch

pytestmark = pytest.mark.gpu
EPS = 2.0 ** -52


@pytest.mark.parametrize("name,nc", [("tiny", 8), ("tiny", 3), ("n400", 13), ("n400", 26), ("n400", 47)])
def test_density_matches_torch(name, nc):
    need_gpu()
    import synth
    s = synth.config_system(name, n_centres=nc, seed=60 + nc)
    pr = problem(s)
    N, A, n = s.N, s.n_aux, pr.n_pairs
    D = dev(np.random.default_rng(nc).standard_normal((N, N)))
    J, K = pr.fock_jk_density(D)
    S = 0.5 * (D + D.T)
    mu, nu = pr.pairs[:n, 0].long(), pr.pairs[:n, 1].long()
    B = torch.zeros((64, N, N), dtype=torch.float64, device="cuda")
    k, k_abs = torch.zeros_like(K), torch.zeros_like(K)
    for p in range(0, A, 64):
        m = min(64, A - p)
        B[:m, mu, nu] = pr.Bc[p:p + m]
        B[:m, nu, mu] = pr.Bc[p:p + m]
        for b, d, out in ((B[:m], S, k), (B[:m].abs(), S.abs(), k_abs)):
            Y = (b.reshape(-1, N) @ d).reshape(m, N, N).permute(1, 0, 2).reshape(N, -1)
            out += 0.5 * Y @ b.reshape(-1, N)
    # a sum of m products is off by at most about m eps times the sum of their magnitudes
    assert bool(((K - k).abs() <= (A * N + 2 * N) * EPS * k_abs).all())
    assert torch.equal(K, K.T) and torch.equal(J, J.T)
    w = torch.where(mu == nu, 1.0, 2.0).double()
    g, g_abs = pr.Bc @ (w * S[mu, nu]), pr.Bc.abs() @ (w * S.abs()[mu, nu])
    assert bool(((J[mu, nu] - pr.Bc.T @ g).abs() <= (n + A) * EPS * (pr.Bc.abs().T @ g_abs)).all())
