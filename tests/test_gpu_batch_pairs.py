"""The batched SCF where its exchange runs over partner lists (N >= 150, sparse enough) beside molecules on packed tiles,
at occupied counts of whole tiles and of quads: each molecule's Fock matrix and energies against the same sums in plain
torch from its own orbitals, the fitted tensor (in FP32 where the exchange reads that) and the oracle's integrals."""
import pytest

import synth
from oracle import integrals as I
from tests.gpu_common import dev, need_gpu, torch

pytestmark = pytest.mark.gpu
EPS, EPS32 = 2.0 ** -52, 2.0 ** -24


def exchange(pr, C, b32, c32):
    """K and the sums of magnitudes, 64 auxiliaries at a time."""
    N, A, n, o = pr.N, pr.n_aux, pr.n_pairs, pr.n_occ
    mu, nu = pr.pairs[:n, 0].long(), pr.pairs[:n, 1].long()
    c = C.float().double() if c32 else C
    K, Ka = (torch.zeros((N, N), dtype=torch.float64, device="cuda") for _ in range(2))
    for p in range(0, A, 64):
        m = min(64, A - p)
        T = pr.T[p:p + m].float().double() if b32 else pr.T[p:p + m]
        B = torch.zeros((m, N, N), dtype=torch.float64, device="cuda")
        B[:, mu, nu] = T
        B[:, nu, mu] = T
        for b, x, out in ((B, c, K), (B.abs(), c.abs(), Ka)):
            X = (b.reshape(-1, N) @ x).reshape(m, N, o).permute(1, 0, 2).reshape(N, -1)
            out += X @ X.T
    return K, Ka


@pytest.mark.parametrize("prec_name,final,graph", [("FP64", False, True), ("FP64", False, False), ("FP32", False, True),
                                                   ("FP32", False, False), ("FP32", True, True)])
def test_fock_and_energy_of_the_last_iteration(prec_name, final, graph):
    need_gpu()
    import paper_2407_19614_amd as P
    from paper_2407_19614_amd.binding import energy_batched, prepare_batch
    prec = getattr(P, prec_name)
    print(f"case: batch over partner lists, {prec_name} final {final} graph {graph}", flush=True)
    systems = [synth.config_system("n400", n_centres=nc, seed=70 + nc) for nc in (27, 14, 15, 33, 17, 16, 40)]
    probs = prepare_batch(systems, prec, workers=2)
    over_lists = [s.N >= 150 and 2 * p.n_pairs - s.N <= 0.6 * s.N ** 2 for s, p in zip(systems, probs)]
    assert sum(over_lists) >= 4 and not all(over_lists)
    tol = dict(tol_E=1e-10, tol_err=1e-8) if prec == P.FP64 else dict(tol_E=1e-7, tol_err=1e-5)
    res, Cs, Fs = energy_batched(probs, prec | (P.FINAL_FP64 if final else 0), want_fock=True, use_graph=graph, **tol)
    for s, pr, r, C, F in zip(systems, probs, res, Cs, Fs):
        assert r["converged"]
        N, A, n, o = s.N, s.n_aux, pr.n_pairs, s.n_occ
        mu, nu = pr.pairs[:n, 0].long(), pr.pairs[:n, 1].long()
        w = torch.where(mu == nu, 1.0, 2.0).double()
        h = dev(I.core_hamiltonian(s))
        D, Da = 2.0 * C @ C.T, 2.0 * C.abs() @ C.abs().T
        # sums of m products are off by at most about m eps times the sum of their magnitudes; in FP32 chains of at
        # most 64 products and one rounding for X and chains of at most 64 rows for K
        g, ga = pr.T @ (w * D[mu, nu]), pr.T.abs() @ (w * Da[mu, nu])
        J, Ja = torch.zeros_like(h), torch.zeros_like(h)
        for M, v in ((J, pr.T.T @ g), (Ja, pr.T.abs().T @ ga)):
            M[mu, nu] = v
            M[nu, mu] = v
        low = prec == P.FP32
        K, Ka = exchange(pr, C, low, low)
        dK = (2 * (64 + 1 + 64) * EPS32 if low else (A * o + 2 * N) * EPS) * Ka
        bound = dK + (n + o + A) * EPS * Ja + 64 * s.n_centres * EPS * h.abs()
        assert bool(((F - (h + J - K)).abs() <= bound).all()), N
        if final:      # the reported energy has the exchange in FP64 arithmetic, from the FP32-stored tensor
            K, Ka = exchange(pr, C, True, False)
            bound = bound - dK + (A * o + 2 * N) * EPS * Ka
        E = float((D * (h + 0.5 * J - 0.5 * K)).sum()) + I.nuclear_repulsion(s)
        size = float((Da * (h.abs() + Ja + Ka)).sum()) + I.nuclear_repulsion(s)
        assert abs(r["E_total"] - E) <= float((Da * bound).sum()) + N * N * EPS * size, N
