"""The gradient with a list that names every pair k times, longer than the room of one auxiliary's products.  With B_c
zero at the repeats and the exchange from the resident B, only the three-centre term depends on k, and is proportional
to it."""
import pytest

import synth
from tests.gpu_common import dev, need_gpu, problem, torch

pytestmark = pytest.mark.gpu


def test_repeated_pairs():
    need_gpu()
    s = synth.config_system("tiny", n_centres=2, seed=9)
    pr = problem(s)
    n, pairs, Bc = pr.n_pairs, pr.pairs.clone(), pr.T.clone()
    C = dev(synth.random_coeffs(s.N, s.n_occ, 3))
    F = dev(synth.random_coeffs(s.N, s.N, 4))

    def gradient(k):
        pr.n_pairs, pr.pairs = k * n, pairs.repeat(k, 1).contiguous()
        pr.T = torch.zeros((s.n_aux, k * n), dtype=torch.float64, device="cuda")
        pr.T[:, :n] = Bc
        return pr.gradient(C, F + F.T)

    k = s.n_aux * s.N ** 2 // n + 1
    assert k * n > s.n_aux * s.N ** 2
    print(f"case: gradient, {n} pairs named {k} times", flush=True)
    one, two, many = gradient(1), gradient(2), gradient(k)
    want = one + (k - 1) * (two - one)
    # FP64 sums of k n_aux n terms
    assert float((many - want).abs().max()) < 1e-12 * k * float(torch.maximum(one.abs(), two.abs()).max())
