"""The setup's kernels at the sizes where they can go wrong: auxiliary counts at and around the 64-row steps of the
factorisation (with the inverse's steps in the same launches) and not a multiple of the 8 that a packing workgroup takes;
an odd N; row counts at and past the 1024 of one pass of the pair offsets' scan."""
import numpy as np
import pytest

from tests.gpu_common import dev, need_gpu, problem, to_np, torch

pytestmark = pytest.mark.gpu

EPS = np.finfo(np.float64).eps


def system(n_fn, n_aux, seed):
    import synth
    xyz = synth.ball_cluster(5, 0.01, 2.5, seed)
    s = synth.make_system(xyz, synth.ORB_BIG, synth.AUX_BIG, tau=1e-12)
    rng = np.random.default_rng(seed)
    s.fn_centre = np.sort(rng.integers(0, 5, n_fn)).astype(np.int32)
    s.fn_exp = rng.uniform(0.1, 20.0, n_fn)
    # widely spread exponents on each centre keep the metric well conditioned
    s.aux_centre = (np.arange(n_aux) % 5).astype(np.int32)
    s.aux_exp = 0.05 * 1.6 ** (np.arange(n_aux) // 5 * 30.0 / (n_aux // 5 + 1))
    s.n_occ = 1
    return s


@pytest.mark.parametrize("n_fn,n_aux", [(7, 1), (33, 63), (64, 64), (65, 65), (129, 127), (31, 130)])
def test_factor_inverse_and_packing(n_fn, n_aux):
    need_gpu()
    pr = problem(system(n_fn, n_aux, n_aux))
    L, Linv = to_np(pr.L), to_np(pr.Linv)
    assert np.all(np.triu(L, 1) == 0.0) and np.all(np.diag(L) > 0.0) and np.all(np.triu(Linv, 1) == 0.0)
    # backward error of a triangular inverse, entry by entry
    assert np.max(np.abs(L @ Linv - np.eye(n_aux)) / (np.abs(L) @ np.abs(Linv) + 1e-300)) < 4 * max(n_aux, 8) * EPS
    nt = (n_fn + 63) // 64
    full = np.zeros((n_aux, 64 * nt, 64 * nt))
    p, Bc = to_np(pr.pairs).astype(int), to_np(pr.Bc)
    full[:, p[:, 0], p[:, 1]] = Bc
    full[:, p[:, 1], p[:, 0]] = Bc
    for prec, dt in ((0, torch.float64), (1, torch.float32)):
        B = to_np(pr.pack_b(prec).view(dt)).reshape(n_aux, nt * (nt + 1) // 2, 64, 64)
        for t, (i, j) in enumerate((i, j) for i in range(nt) for j in range(i + 1)):
            want = full[:, 64 * i:64 * i + 64, 64 * j:64 * j + 64].astype(B.dtype)
            assert np.array_equal(B[:, t], want)


@pytest.mark.parametrize("n_fn", [1, 1023, 1024, 1025, 2049])
def test_pair_list(n_fn):
    need_gpu()
    import paper_2407_19614_amd as P
    s = system(n_fn, 5, 3)
    s.fn_exp = np.tile([0.2, 40.0, 900.0], n_fn)[:n_fn]      # many pairs of different centres drop out
    pr = P.RIProblem(s, device="cuda", prec=P.FP64)
    n = pr.build_3c()
    p = to_np(pr.pairs)[:n].astype(np.int64)
    i, j = np.tril_indices(n_fn)
    a, b = s.fn_exp[i], s.fn_exp[j]
    r2 = ((s.xyz[s.fn_centre[i]] - s.xyz[s.fn_centre[j]]) ** 2).sum(-1)
    k = (4 * a * b / np.pi ** 2) ** 0.75 * np.exp(-a * b / (a + b) * r2)
    q = k * k * 2 * np.pi ** 2.5 / ((a + b) ** 2 * np.sqrt(2 * (a + b)))
    keep = q > s.tau * (1 - 1e-9)
    assert np.array_equal(keep, q > s.tau * (1 + 1e-9))       # no pair within rounding of the threshold
    assert np.array_equal(p, np.stack([i[keep], j[keep]], 1))
