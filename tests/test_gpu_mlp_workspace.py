"""The network's calls write nothing past the workspace that ri_workspace_bytes asks for: an exactly sized workspace
inside a larger buffer with a pattern on both sides, at row counts where the last split of the weight gradient is short
(one block past a multiple of 2048 rows) and around the block sizes."""
import ctypes

import numpy as np
import pytest

from oracle import mlp as M
from tests.gpu_common import need_gpu, to_np, torch

pytestmark = pytest.mark.gpu
GUARD = 1 << 20


@pytest.mark.parametrize("n", [1, 2049, 8192, 8193, 8256, 8257, 10304, 16385, 16384 + 64])
def test_calls_stay_inside_their_workspace(n):
    need_gpu()
    import paper_2407_19614_amd as P
    from paper_2407_19614_amd import binding as Bd
    print(f"case: network workspace, {n} rows", flush=True)
    rng = np.random.default_rng(n)
    net = P.MLP(P.pack_params(M.init_params(seed=n)), np.zeros(8, np.float32), np.ones(8, np.float32))
    feat = torch.tensor(rng.normal(0, 1, (n, 8)).astype(np.float32), device="cuda")
    t = torch.tensor(rng.normal(0, 0.3, n).astype(np.float32), device="cuda")
    pp = P.unpack_params(to_np(net.params))
    nb = Bd.workspace_bytes(Bd.OP_MLP, 1, 1, 1, n, P.FP64)
    buf = torch.full((nb + 2 * GUARD,), 0xA5, dtype=torch.uint8, device="cuda")
    ws = ctypes.c_void_p(buf.data_ptr() + GUARD)
    p = lambda x: ctypes.c_void_p(x.data_ptr())
    y, loss, g = torch.empty(n, device="cuda"), torch.empty(1, device="cuda"), torch.empty_like(net.params)
    for prec in (P.MLP_FP32, P.MLP_BF16):
        assert P.lib().ri_mlp_forward(ctypes.byref(net.c), p(feat), n, p(y), prec, ws, nb, net.stream()) == 0
    assert P.lib().ri_mlp_train_step(ctypes.byref(net.c), p(net.m), p(net.v), 1, 1e-3, p(feat), p(t), n, p(loss), p(g),
                                     ws, nb, net.stream()) == 0
    torch.cuda.synchronize()
    assert bool((buf[:GUARD] == 0xA5).all()) and bool((buf[GUARD + nb:] == 0xA5).all())
    # FP32 sums: the tolerance of the row-count test
    _, gref = M.loss_and_grad(pp, feat.cpu().numpy().astype(np.float64), t.cpu().numpy().astype(np.float64))
    gv = P.unpack_params(to_np(g))
    for k in gref:
        assert np.abs(gv[k] - gref[k]).max() < 1e-4 * np.abs(gref[k]).max() + 1e-9, k
