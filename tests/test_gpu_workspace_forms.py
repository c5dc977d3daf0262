"""X over the partner lists against X from packed tiles on the same inputs.  The form follows from the room in the
workspace: one that is short of the lists is taken for the packed form.  FP32 results are
the same bits in both forms (zeros left out of a chain of fused multiply-adds change nothing); FP64 ones agree to
rounding."""
import ctypes

import pytest

from tests.gpu_common import dev, need_gpu, problem, torch

pytestmark = pytest.mark.gpu
EPS = 2.0 ** -52


def _system(nc, n_occ):
    import synth
    s = synth.config_system("n400", n_centres=nc, seed=90 + nc)
    s.n_occ = n_occ
    return s


def _packed_only(pr, op, prec):
    """One byte less than the lists need."""
    from paper_2407_19614_amd import binding as Bd
    nb = Bd.workspace_bytes(op, pr.N, pr.n_aux, pr.n_occ, pr.n_pairs, prec) - 1
    return torch.empty(nb, dtype=torch.uint8, device="cuda"), nb


def _p(t):
    return None if t is None else ctypes.c_void_p(t.data_ptr())


@pytest.mark.parametrize("prec_name,nc,n_occ", [("FP64", 37, 37), ("FP64", 31, 128), ("FP32", 40, 40), ("FP32", 37, 133),
                                                ("FP32", 44, 100)])
def test_fock_build(prec_name, nc, n_occ):
    need_gpu()
    import paper_2407_19614_amd as P
    from paper_2407_19614_amd import binding as Bd
    import synth
    prec = getattr(P, prec_name)
    print(f"case: both forms of X, {prec_name}, {nc} centres, {n_occ} occupied", flush=True)
    pr = problem(_system(nc, n_occ), prec)
    C = dev(synth.random_coeffs(pr.N, n_occ, 5))
    J0, K0, g0 = pr.fock_jk(C)
    ws, nb = _packed_only(pr, Bd.OP_FOCK, prec)
    J1, K1, g1 = torch.empty_like(J0), torch.empty_like(K0), torch.empty_like(g0)
    assert P.lib().ri_fock_jk(pr.N, pr.n_aux, n_occ, _p(pr.B), prec, _p(pr.T), _p(pr.pairs), pr.n_pairs, _p(C), _p(J1),
                              _p(K1), _p(g1), _p(ws), nb, pr.stream()) == 0
    torch.cuda.synchronize()
    if prec == P.FP32:
        assert torch.equal(K0, K1) and torch.equal(J0, J1) and torch.equal(g0, g1)
        return
    # K: a diagonal entry is a sum of n_aux n_occ squares, and |K_mn| <= sqrt(K_mm K_nn); each X is off by at most N
    # roundings of a sum whose terms may cancel, so compare with the sums of magnitudes
    mu, nu = pr.pairs[:pr.n_pairs, 0].long(), pr.pairs[:pr.n_pairs, 1].long()
    k_abs = torch.zeros_like(K0)
    for p in range(0, pr.n_aux, 64):
        m = min(64, pr.n_aux - p)
        B = torch.zeros((m, pr.N, pr.N), dtype=torch.float64, device="cuda")
        B[:, mu, nu] = pr.T[p:p + m].abs()
        B[:, nu, mu] = pr.T[p:p + m].abs()
        X = (B.reshape(-1, pr.N) @ C.abs()).reshape(m, pr.N, n_occ).permute(1, 0, 2).reshape(pr.N, -1)
        k_abs += X @ X.T
    assert bool(((K0 - K1).abs() <= 2 * (pr.n_aux * n_occ + 2 * pr.N) * EPS * k_abs).all())
    w = torch.where(mu == nu, 1.0, 2.0).double()
    j_abs = pr.T.abs().T @ (pr.T.abs() @ (w * (2.0 * C.abs() @ C.abs().T)[mu, nu]))
    assert bool(((J0 - J1)[mu, nu].abs() <= 2 * (pr.n_pairs + n_occ + pr.n_aux) * EPS * j_abs).all())


@pytest.mark.parametrize("prec_name,final", [("FP64", False), ("FP32", False), ("FP32", True), ("BF16X6", True)])
def test_scf_and_gradient(prec_name, final):
    need_gpu()
    import paper_2407_19614_amd as P
    from paper_2407_19614_amd import binding as Bd
    prec = getattr(P, prec_name)
    print(f"case: both forms of X in the SCF and the gradient, {prec_name} final {final}", flush=True)
    pr = problem(_system(44, 44), prec)
    arg = prec | (P.FINAL_FP64 if final else 0)
    r0, C0, F0, _ = pr.energy(max_iter=60, tol_E=1e-8, tol_err=1e-5, final_fp64=final)
    ws, nb = _packed_only(pr, Bd.OP_ENERGY, arg)
    opts, r1 = Bd.SCFOpts(60, 6, 1e-8, 1e-5, 0, 0), Bd.SCFResult()
    C1, F1 = torch.empty_like(C0), torch.empty_like(F0)
    assert P.lib().ri_energy(ctypes.byref(pr.c_sys), _p(pr.B), arg, _p(pr.T), _p(pr.pairs), pr.n_pairs, ctypes.byref(opts),
                             None, _p(C1), _p(F1), None, ctypes.byref(r1), _p(ws), nb, pr.stream()) == 0
    assert r1.n_iter == r0["n_iter"]
    if prec == P.FP64:
        # both stop at an energy change below 1e-8 on the same path
        assert abs(r1.E_total - r0["E_total"]) < 1e-8
    else:
        # the iterations are the same bits; the FP64 build at the end sums n_aux n_occ N^2 terms of size E in another order
        assert torch.equal(C0, C1) and torch.equal(F0, F1)
        assert abs(r1.E_total - r0["E_total"]) <= (0.0 if not final else 1e-10 * abs(r0["E_total"]))
    ws, nb = _packed_only(pr, Bd.OP_GRADIENT, prec)
    g0, g1 = pr.gradient(C0, F0), torch.empty((pr.system.n_centres, 3), dtype=torch.float64, device="cuda")
    assert P.lib().ri_gradient(ctypes.byref(pr.c_sys), _p(pr.pairs), pr.n_pairs, _p(pr.B), prec, _p(pr.T), _p(pr.Linv),
                               _p(C0), _p(F0), _p(g1), _p(ws), nb, pr.stream()) == 0
    torch.cuda.synchronize()
    # sums over all pairs and auxiliaries by atomic adds; Xi carries the metric's condition
    assert float((g0 - g1).abs().max()) < 1e-9 * max(1.0, float(g0.abs().max()))


@pytest.mark.parametrize("prec_name", ["FP64", "FP32"])
def test_compressed_calls_hold_no_slab_beside_the_lists(prec_name):
    need_gpu()
    import paper_2407_19614_amd as P
    from paper_2407_19614_amd import binding as Bd
    prec = getattr(P, prec_name)
    print(f"case: compressed over the lists, {prec_name}", flush=True)
    s = _system(44, 44)
    out = []
    for comp in (False, True):
        pr = P.RIProblem(s, prec=prec, compressed=comp)
        pr.build_3c()
        pr.metric_factor(prec)
        r, C, F, _ = pr.energy(max_iter=60, tol_E=1e-8, tol_err=1e-5)
        out.append((r["E_total"], C, F, *pr.fock_jk(C), pr.gradient(C, F)))
    assert out[0][0] == out[1][0] and all(torch.equal(a, b) for a, b in zip(out[0][1:-1], out[1][1:-1]))
    assert float((out[0][-1] - out[1][-1]).abs().max()) < 1e-9 * max(1.0, float(out[0][-1].abs().max()))
    most = max(Bd.workspace_bytes(op, s.N, s.n_aux, s.n_occ, pr.n_pairs, prec)
               for op in (Bd.OP_FOCK, Bd.OP_ENERGY, Bd.OP_GRADIENT))
    assert pr._ws.numel() <= most
