"""The compressed form where X is formed slab by slab from packed tiles: several slabs with a ragged last one, in a build
too small for the partner lists and in larger ones with too many pairs for them (in FP32 the compressed form alone takes
lists at half of the pairs).  Equal to the resident form bit for bit and to plain torch in FP64 within rounding."""
import pytest

import synth
from tests.gpu_common import dev, need_gpu, torch

pytestmark = pytest.mark.gpu


# N = 10 nc, 30 nc auxiliaries; tau 0: every pair, 1e-25: about half of them
@pytest.mark.parametrize("nc,n_occ,tau", [(21, 21, None), (31, 47, 0.0), (31, 130, 0.0), (39, 39, 1e-25)])
@pytest.mark.parametrize("prec_name", ["FP64", "FP32"])
def test_slabs(prec_name, nc, n_occ, tau):
    need_gpu()
    import paper_2407_19614_amd as P
    from paper_2407_19614_amd import binding as Bd
    prec = getattr(P, prec_name)
    print(f"case: compressed slabs, {prec_name} {nc} centres {n_occ} occupied", flush=True)
    s = synth.config_system("n400", n_centres=nc, seed=110 + nc)
    s.n_occ = n_occ
    assert s.n_aux > 2 * Bd.COMPRESSED_SLAB and s.n_aux % Bd.COMPRESSED_SLAB != 0
    C = dev(synth.random_coeffs(s.N, n_occ, seed=5))
    F = dev(synth.random_coeffs(s.N, s.N, seed=6))
    out = []
    for comp in (False, True):
        pr = P.RIProblem(s, prec=prec, compressed=comp)
        pr.build_3c(tau=tau)
        pr.metric_factor(prec)
        out.append((*pr.fock_jk(C), pr.gradient(C, F + F.T)))
    N, A, n = s.N, s.n_aux, pr.n_pairs
    pad, fill = (N + 127) // 128 * 128, (2 * n - N) / N ** 2
    assert (A * n_occ + 31) * pad * 8 <= 64 << 20 or (fill > 0.6 if tau == 0.0 else 0.42 < fill < 0.6)
    assert all(torch.equal(a, b) for a, b in zip(out[0][:3], out[1][:3]))
    g0, g1 = out[0][3], out[1][3]      # sums over centres by atomic adds
    assert float((g0 - g1).abs().max()) < 1e-10 * float(g0.abs().max())
    K = out[1][1]
    mu, nu = pr.pairs[:n, 0].long(), pr.pairs[:n, 1].long()
    low = prec == P.FP32
    c = C.float().double() if low else C
    k, k_abs = torch.zeros_like(K), torch.zeros_like(K)
    for p in range(0, A, 64):
        m = min(64, A - p)
        T = pr.T[p:p + m].float().double() if low else pr.T[p:p + m]
        B = torch.zeros((m, N, N), dtype=torch.float64, device="cuda")
        B[:, mu, nu] = T
        B[:, nu, mu] = T
        for b, x, o in ((B, c, k), (B.abs(), c.abs(), k_abs)):
            X = (b.reshape(-1, N) @ x).reshape(m, N, n_occ).permute(1, 0, 2).reshape(N, -1)
            o += X @ X.T
    # a sum of m products is off by at most about m eps times the sum of their magnitudes; in FP32 chains of at most 64
    # products and one rounding for X and chains of at most 64 rows for K
    bound = 2 * (64 + 1 + 64) * 2.0 ** -24 if low else (A * n_occ + 2 * N) * 2.0 ** -52
    assert bool(((K - k).abs() <= bound * k_abs).all())
