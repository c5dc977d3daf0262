"""The FP32 gradient uses both halves of each B_ij^P.  The half-transform's C is rounded to FP32 and the other C of
C^T B^P C is not, so for orbitals that FP32 does not hold exactly the two halves differ by a known amount; everything else
of this input (multiples of 1/8 in B, an identity metric factor) is exact in FP32.  The reference forms the same sums in
64 bits from the mean of the halves."""
import numpy as np
import pytest

import synth
from oracle import integrals as I
from tests.gpu_common import dev, need_gpu, to_np, torch

pytestmark = pytest.mark.gpu


def reference(s, mu, nu, Bc, C, Bij):
    n, na = s.n_occ, s.n_aux
    w = np.where(mu == nu, 1.0, 2.0)
    D = 2.0 * C @ C.T
    c = Bc @ (w * D[mu, nu])
    fc, g, size = s.fn_centre, np.zeros_like(s.xyz), 0.0
    dS, dT = I.overlap_kinetic_derivs(s)
    vA, vB, vC = I.nuclear_derivs(s)
    np.add.at(g, np.repeat(fc, s.N), (D[..., None] * (dT + vA)).reshape(-1, 3))
    np.add.at(g, np.tile(fc, s.N), (D[..., None] * (-dT + vB)).reshape(-1, 3))
    g += np.einsum("mn,cmnx->cx", D, vC)
    for P in range(na):
        dA, dB = I.eri3_derivs_pairs(s, mu, nu, [P])
        Y = w * (c[P] * D - 2.0 * C @ Bij[P] @ C.T)[mu, nu]
        cA, cB = Y[:, None] * dA[0], Y[:, None] * dB[0]
        np.add.at(g, fc[mu], cA)
        np.add.at(g, fc[nu], cB)
        g[s.aux_centre[P]] -= cA.sum(0) + cB.sum(0)
        size += np.abs(cA).sum() + np.abs(cB).sum()
    X = Bij.reshape(na, n * n)
    t = (-0.5 * (np.outer(c, c) - 2.0 * X @ X.T))[..., None] * I.metric_derivs(s)
    np.add.at(g, s.aux_centre, t.sum(1))
    np.add.at(g, s.aux_centre, -t.sum(0))
    return g + I.nuclear_repulsion_grad(s), size + 2 * np.abs(t).sum()


@pytest.mark.parametrize("nc,n_occ", [(3, 2), (8, 5), (8, 17)])
def test_both_halves_enter(nc, n_occ):
    need_gpu()
    import paper_2407_19614_amd as P
    s = synth.config_system("tiny", n_centres=nc, seed=40 + nc)
    s.n_occ = n_occ
    print(f"case: FP32 gradient, {nc} centres, {n_occ} occupied", flush=True)
    pr = P.RIProblem(s, prec=P.FP32)
    pr.build_3c()
    pr.metric_factor(P.FP32)
    rng = np.random.default_rng(nc)
    mu, nu = (to_np(pr.pairs)[: pr.n_pairs, k].astype(np.int64) for k in (0, 1))
    Bc = rng.integers(-8, 9, (s.n_aux, pr.n_pairs)) / 8.0
    # columns of C alternate between multiples of 1/8 and the same times 1 + 2^-26, which rounds back
    Cr = rng.integers(-8, 9, (s.N, n_occ)) / 8.0
    f = np.where(np.arange(n_occ) % 2 == 1, 1.0 + 2.0 ** -26, 1.0)
    C = Cr * f
    assert np.array_equal(C.astype(np.float32).astype(np.float64), Cr)
    pr.T = dev(Bc)
    pr.B = pr.pack_b(P.FP32)
    pr.Linv = torch.eye(s.n_aux, dtype=torch.float64, device="cuda")
    got = to_np(pr.gradient(dev(C), torch.zeros((s.N, s.N), dtype=torch.float64, device="cuda")))
    B = np.zeros((s.n_aux, s.N, s.N))
    B[:, mu, nu] = Bc
    B[:, nu, mu] = Bc
    half = np.einsum("pmn,mi,nj->pij", B, Cr, C, optimize=True)   # [P][i][j]: i through FP32
    both = 0.5 * (half + half.transpose(0, 2, 1))
    lower = np.tril(half) + np.tril(half, -1).transpose(0, 2, 1)
    want, size = reference(s, mu, nu, Bc, C, both)
    one_half, _ = reference(s, mu, nu, Bc, C, lower)
    # FP64 sums of at most n_aux n_pairs terms; the Boys functions and the other terms at 1e-14 of theirs
    tol = 1e-13 * size
    assert np.abs(one_half - want).max() > 20 * tol               # the input tells the two apart
    assert np.abs(got - want).max() < tol


# packed halves: occupied counts around the 32-wide tiles, sizes past the switch from whole blocks
@pytest.mark.parametrize("nc,n_occ", [(21, 33), (20, 64), (20, 97), (13, 130)])
def test_packed_halves_match_fp64(nc, n_occ):
    need_gpu()
    import paper_2407_19614_amd as P
    print(f"case: FP32 gradient with packed halves, {nc} centres, {n_occ} occupied", flush=True)
    s = synth.config_system("n400", n_centres=nc, seed=nc)
    s.n_occ = n_occ
    assert s.n_aux ** 2 * n_occ ** 2 >= 4e8
    C, F = dev(synth.random_coeffs(s.N, n_occ, 3)), dev(synth.random_coeffs(s.N, s.N, 4))
    g = []
    for prec in (P.FP64, P.FP32):
        pr = P.RIProblem(s, prec=prec)
        pr.build_3c()
        pr.metric_factor(prec)
        g.append(pr.gradient(C, F + F.T))
    # B and one C rounded to FP32, X to FP32 after sums of at most N products: 3 + log2 N roundings of 2^-24 on terms
    # that cancel by up to 1e3 in the components' sums
    assert float((g[0] - g[1]).norm() / g[0].norm()) < 11 * 2.0 ** -24 * 1e3
