"""The gradient at the most centres it takes: centres without charge and functions between those of a small molecule
change nothing and have no force of their own."""
import numpy as np
import pytest

import synth
from tests.gpu_common import dev, need_gpu, problem, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nc", [300, 2047, 2048])
def test_empty_centres(nc):
    need_gpu()
    print(f"case: gradient with {nc} centres", flush=True)
    s = synth.config_system("tiny")
    rng = np.random.default_rng(nc)
    at = np.sort(rng.choice(nc, s.n_centres, replace=False)).astype(np.int32)
    at[-1] = nc - 1
    xyz = rng.uniform(50.0, 90.0, (nc, 3))
    xyz[at] = s.xyz
    Z = np.zeros(nc)
    Z[at] = s.Z
    big = synth.System(xyz, Z, at[s.fn_centre], s.fn_exp, at[s.aux_centre], s.aux_exp, s.n_occ, s.tau)
    C = dev(synth.random_coeffs(s.N, s.n_occ, 3))
    F = dev(synth.random_coeffs(s.N, s.N, 4))
    want = to_np(problem(s).gradient(C, F + F.T))
    got = to_np(problem(big).gradient(C, F + F.T))
    rest = np.ones(nc, bool)
    rest[at] = False
    assert np.all(got[rest] == 0.0)
    # the same terms in another order of atomic adds
    assert np.abs(got[at] - want).max() < 1e-12 * np.abs(want).max()
