"""The SCF's density start where its Fock build has less room than a build of its own (several slabs, ragged last ones):
the first iteration against one started from the occupied orbitals of the same Fock matrix, formed from the separate
density build."""
import numpy as np
import pytest

import synth
from oracle import integrals as I
from tests.gpu_common import dev, need_gpu, problem, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,nc,prec_name", [("tiny", 8, "FP64"), ("n400", 13, "FP64"), ("n400", 13, "FP32"),
                                               ("n400", 27, "FP64"), ("n400", 33, "FP32"), ("n400", 33, "FP64")])
def test_first_iteration(name, nc, prec_name):
    need_gpu()
    import scipy.linalg as sla
    import paper_2407_19614_amd as P
    print(f"case: density start, {name} {nc} centres {prec_name}", flush=True)
    s = synth.config_system(name, n_centres=nc, seed=20 + nc)
    pr = problem(s, getattr(P, prec_name))
    C0 = pr.energy(max_iter=3, raise_on_noconv=False)[1]
    D = 2.0 * C0 @ C0.T
    J, K = pr.fock_jk_density(D)
    r, C, F, _ = pr.energy(max_iter=1, raise_on_noconv=False, guess_density=D, density_fock=True)
    h, S = I.core_hamiltonian(s), I.overlap(s)
    w, V = sla.eigh(h + to_np(J) - to_np(K), S)
    assert w[s.n_occ] - w[s.n_occ - 1] > 1e-2
    r1, C1, F1, _ = pr.energy(max_iter=1, raise_on_noconv=False, guess=dev(V[:, : s.n_occ]))
    # the occupied spaces agree to rounding over the gap times the condition of S; E is stationary in neither, so first order
    tol = 1e-14 * np.linalg.cond(S) * np.abs(w).max() / (w[s.n_occ] - w[s.n_occ - 1])
    if prec_name == "FP32":
        tol = max(tol, 1e-5)     # different orbitals of one space, each rounded to FP32
    assert abs(r["E_total"] - r1["E_total"]) <= max(tol, 1e-12) * abs(r1["E_total"])
