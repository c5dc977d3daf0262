"""The gradient where the products at the pairs change shape: occupied counts around the 64 that switch the auxiliaries
a wave takes and the 128 of one launch, odd rows of partners; against the same formula in plain torch with automatic
differentiation of the integrals."""
import math

import pytest

from tests.gpu_common import dev, need_gpu, problem, torch

pytestmark = pytest.mark.gpu


def boys(t):
    small = t < 1.0
    u = torch.where(small, t, torch.zeros_like(t))
    f = torch.zeros_like(t)
    for k in range(20, -1, -1):
        f = f * u + (-1.0) ** k / (math.factorial(k) * (2 * k + 1))
    r = torch.sqrt(torch.where(small, torch.ones_like(t), t))
    return torch.where(small, f, 0.5 * math.sqrt(math.pi) * torch.erf(r) / r)


@pytest.mark.parametrize("name,nc,n_occ", [("tiny", 3, 5), ("tiny", 8, 8), ("n400", 10, 47), ("n400", 17, 65),
                                           ("n400", 17, 128), ("n400", 17, 137), ("n400", 31, 31)])
def test_gradient_of_given_orbitals(name, nc, n_occ):
    need_gpu()
    import synth
    s = synth.config_system(name, n_centres=nc, seed=30 + nc)
    s.n_occ = n_occ
    pr = problem(s)
    N, A, n, o = s.N, s.n_aux, pr.n_pairs, n_occ
    C = dev(synth.random_coeffs(N, o, 3))
    F = dev(synth.random_coeffs(N, N, 4))
    F = F + F.T
    got = pr.gradient(C, F)
    fc, ac = dev(s.fn_centre).long(), dev(s.aux_centre).long()
    fe, ae, Z = dev(s.fn_exp), dev(s.aux_exp), dev(s.Z)
    mu, nu = pr.pairs[:n, 0].long(), pr.pairs[:n, 1].long()
    w = torch.where(mu == nu, 1.0, 2.0).double()
    norm = lambda a: (2 * a / math.pi) ** 0.75
    D = 2 * C @ C.T
    W = 0.5 * D @ F @ D
    d = w * D[mu, nu]
    L = pr.Linv
    Bc = pr.Bc
    Bij = torch.empty((A, o * o), dtype=torch.float64, device="cuda")
    for P in range(A):
        B = torch.zeros((N, N), dtype=torch.float64, device="cuda")
        B[mu, nu] = Bc[P]
        B[nu, mu] = Bc[P]
        Bij[P] = (C.T @ B @ C).reshape(-1)
    Xi, c = L.T @ Bij, L.T @ (Bc @ d)
    Zm = c[:, None] * c[None] - 2 * Xi @ Xi.T
    Y = torch.empty((A, n), dtype=torch.float64, device="cuda")
    for P in range(A):
        Y[P] = w * (c[P] * D[mu, nu] - 2 * (C @ Xi[P].reshape(o, o) @ C.T)[mu, nu])
    x = dev(s.xyz).requires_grad_(True)

    def gauss(i, j):
        a, b = fe[i], fe[j]
        p = a + b
        r2 = ((x[fc[i]] - x[fc[j]]) ** 2).sum(-1)
        return p, (a[:, None] * x[fc[i]] + b[:, None] * x[fc[j]]) / p[:, None], norm(a) * norm(b) * torch.exp(-a * b / p * r2), a * b / p, r2

    i, j = torch.tril_indices(N, N, device="cuda")
    ww = torch.where(i == j, 1.0, 2.0).double()
    p, G, k, r, r2 = gauss(i, j)
    S = k * (math.pi / p) ** 1.5
    h = S * r * (3 - 2 * r * r2)
    for q in range(s.n_centres):
        h = h - Z[q] * k * 2 * math.pi / p * boys(p * ((G - x[q]) ** 2).sum(-1))
    e = (ww * D[i, j] * h).sum() - (ww * W[i, j] * S).sum()
    p, G, k, _, _ = gauss(mu, nu)
    cc = ae[:, None]
    T = k * norm(cc) * 2 * math.pi ** 2.5 / (p * cc * torch.sqrt(p + cc)) * boys(
        p * cc / (p + cc) * ((G[None] - x[ac][:, None]) ** 2).sum(-1))
    e = e + (Y * T).sum()
    a, b = ae[:, None], ae[None]
    M = norm(a) * norm(b) * 2 * math.pi ** 2.5 / (a * b * torch.sqrt(a + b)) * boys(
        a * b / (a + b) * ((x[ac][:, None] - x[ac][None]) ** 2).sum(-1))
    e = e - 0.5 * (Zm * M).sum()
    i, j = torch.triu_indices(s.n_centres, s.n_centres, 1, device="cuda")
    e = e + (Z[i] * Z[j] / (x[i] - x[j]).norm(dim=-1)).sum()
    ref, = torch.autograd.grad(e, x)
    # random orbitals and F: the terms are large and cancel; Xi carries the metric's condition
    scale = float((Y.abs() * T.detach().abs()).sum() / s.n_centres + (Zm.abs() * M.detach().abs()).sum() / s.n_centres)
    assert float((got - ref).abs().max()) < 1e-9 * max(scale, 1.0)
