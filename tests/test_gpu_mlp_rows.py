"""The network's launches at the row counts where their blocks end: one row, around 32 (small blocks) and 64, on both
sides of the switch to 64-row blocks, and counts whose last split of the weight gradient is short; against the oracle."""
import numpy as np
import pytest

from oracle import mlp as M
from tests.gpu_common import need_gpu, to_np, torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 31, 33, 100, 2049, 8192, 8193, 16384 + 5])
def test_rows(n):
    need_gpu()
    import paper_2407_19614_amd as P
    rng = np.random.default_rng(n)
    p = M.init_params(seed=n)
    for k in ("b1", "b2", "b3"):
        p[k] = rng.normal(0, 0.1, p[k].shape)
    mu, sg = rng.normal(0, 1, 8).astype(np.float32), rng.uniform(0.5, 2, 8).astype(np.float32)
    feat = rng.normal(0, 1, (n, 8)).astype(np.float32)
    t = rng.normal(0, 0.3, n).astype(np.float32)
    pp = P.unpack_params(P.pack_params(p))
    x = (feat.astype(np.float64) - mu) / sg
    yref, _ = M.forward(pp, x)
    net = P.MLP(P.pack_params(p), mu, sg)
    f = torch.tensor(feat, device="cuda")
    scale = np.abs(yref).max()
    # FP32 sums of 256 terms: 256 * 2^-24 of their magnitude; BF16 operands: 2^-8 of it
    assert np.abs(to_np(net.forward(f, P.MLP_FP32)) - yref).max() < 3e-5 * max(scale, 1)
    assert np.abs(to_np(net.forward(f, P.MLP_BF16)) - yref).max() < 3e-2 * max(scale, 1)
    loss, g = net.train_step(f, torch.tensor(t, device="cuda"), lr=1e-3, want_grad=True)
    lref, gref = M.loss_and_grad(pp, x, t.astype(np.float64))
    assert abs(float(to_np(loss)[0]) - lref) < 1e-4 * lref
    gv = P.unpack_params(to_np(g))
    for k in gref:
        assert np.abs(gv[k] - gref[k]).max() < 1e-4 * np.abs(gref[k]).max() + 1e-9, k
    again, g2 = P.MLP(P.pack_params(p), mu, sg).train_step(f, torch.tensor(t, device="cuda"), lr=1e-3, want_grad=True)
    assert torch.equal(g, g2) and torch.equal(loss, again)
