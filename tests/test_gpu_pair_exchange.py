"""J and K where the exchange runs over each row's significant partners (screened systems
whose X^T is over 64 MiB), against plain torch in FP64 from the same fitted tensor."""
import numpy as np
import pytest

from gpu_common import dev, need_gpu, problem

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
EPS = 2.0 ** -52


# centres (N = 10 per centre, 30 auxiliaries), occupied rows: one tile and quads, whole tiles,
# a padded last tile, over one and over two chunks of 128, the sizes beside the 64 MiB rule
@pytest.mark.parametrize("nc,n_occ", [(27, 27), (26, 26), (28, 64), (31, 47), (31, 128), (29, 133), (27, 270)])
def test_pair_exchange_matches_torch(nc, n_occ):
    need_gpu()
    import synth
    s = synth.config_system("n400", n_centres=nc, seed=50 + nc)
    s.n_occ = n_occ
    pr = problem(s)
    C = dev(synth.random_coeffs(s.N, n_occ, 7))
    J, K, gamma = pr.fock_jk(C)
    N, A, n = s.N, s.n_aux, pr.n_pairs
    mu, nu = pr.pairs[:n, 0].long(), pr.pairs[:n, 1].long()
    assert 0 < 2 * n - N <= 0.6 * N * N
    w = torch.where(mu == nu, 1.0, 2.0).double()
    D = 2.0 * C @ C.T
    d = w * D[mu, nu]
    g = pr.Bc @ d
    # each sum of m products is off by at most about m eps times the sum of their magnitudes
    da = w * (2.0 * C.abs() @ C.abs().T)[mu, nu]
    g_abs = pr.Bc.abs() @ da
    assert bool(((gamma - g).abs() <= (n + n_occ) * EPS * g_abs).all())
    j, j_abs = pr.Bc.T @ g, pr.Bc.abs().T @ g_abs
    assert bool(((J[mu, nu] - j).abs() <= (n + n_occ + A) * EPS * j_abs).all())
    assert torch.equal(J, J.T) and torch.equal(K, K.T)
    B = torch.zeros((64, N, N), dtype=torch.float64, device="cuda")
    k, k_abs = torch.zeros_like(K), torch.zeros_like(K)
    for p in range(0, A, 64):
        m = min(64, A - p)
        B[:m, mu, nu] = pr.Bc[p:p + m]
        B[:m, nu, mu] = pr.Bc[p:p + m]
        for b, c, out in ((B, C, k), (B.abs(), C.abs(), k_abs)):
            X = (b[:m].reshape(-1, N) @ c).reshape(m, N, n_occ).permute(1, 0, 2).reshape(N, -1)
            out += X @ X.T
    assert bool(((K - k).abs() <= (A * n_occ + 2 * N) * EPS * k_abs).all())
    # entries off the significant pairs get no J
    off = torch.ones((N, N), dtype=torch.bool, device="cuda")
    off[mu, nu] = False
    off[nu, mu] = False
    assert bool((J[off] == 0).all())


def test_pair_exchange_is_reproducible():
    need_gpu()
    import synth
    s = synth.config_system("n400", n_centres=31, seed=3)
    pr = problem(s)
    C = dev(synth.random_coeffs(s.N, s.n_occ, 7))
    first = pr.fock_jk(C)
    again = pr.fock_jk(C)
    assert all(torch.equal(a, b) for a, b in zip(first, again))
    assert np.isfinite(first[1].cpu().numpy()).all()


# FP32 over the partner lists is the dense FP32 kernel's arithmetic: per 64 nu one chain of
# fused multiply-adds in ascending nu (zeros change nothing), added in FP64
@pytest.mark.parametrize("nc,n_occ", [(40, 40), (37, 47), (44, 100), (38, 128), (37, 133)])
def test_pair_exchange_fp32_error(nc, n_occ):
    need_gpu()
    import paper_2407_19614_amd as P
    import synth
    s = synth.config_system("n400", n_centres=nc, seed=70 + nc)
    s.n_occ = n_occ
    C = dev(synth.random_coeffs(s.N, n_occ, 9))
    pr = problem(s, P.FP32)
    N, A, n = s.N, s.n_aux, pr.n_pairs
    assert A * n_occ * ((N + 127) // 128 * 128) * 4 > 64 << 20 and 2 * n - N <= 0.6 * N * N
    K = pr.fock_jk(C)[1]
    mu, nu = pr.pairs[:n, 0].long(), pr.pairs[:n, 1].long()
    B = torch.zeros((64, N, N), dtype=torch.float32, device="cuda")
    c32 = C.float()
    k, k_abs = torch.zeros_like(K), torch.zeros_like(K)
    for p in range(0, A, 64):
        m = min(64, A - p)
        B[:m, mu, nu] = pr.Bc[p:p + m].float()
        B[:m, nu, mu] = pr.Bc[p:p + m].float()
        b = B[:m].double()
        X = (b.reshape(-1, N) @ c32.double()).reshape(m, N, n_occ).permute(1, 0, 2).reshape(N, -1)
        Xa = (b.abs().reshape(-1, N) @ c32.double().abs()).reshape(m, N, n_occ).permute(1, 0, 2).reshape(N, -1)
        k += X @ X.T
        k_abs += Xa @ Xa.T
    # X: chains of at most 64 products and one rounding to FP32; K: chains of at most 64 rows
    assert bool(((K - k).abs() <= 2 * (64 + 1 + 64) * 2.0 ** -24 * k_abs).all())
