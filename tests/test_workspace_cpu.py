"""A workspace sized for a longer pair list is enough for every shorter one, without a GPU: the calls get past their size
check and fail at the HIP runtime, before anything is read."""
import ctypes

import pytest

import paper_2407_19614_amd as P
from paper_2407_19614_amd import binding as Bd

WORKSPACE, HIP = 4, 6


def _call(op, N, na, no, n_pairs, prec, nb):
    d = ctypes.create_string_buffer(1 << 12)         # stands in for device memory; never read
    p = ctypes.cast(d, ctypes.c_void_p)
    s = Bd.RISystem(N // 10, N, na, no, *[ctypes.cast(d, ctypes.c_void_p).value] * 6)
    B = None if prec & P.COMPRESSED else p
    if op == Bd.OP_FOCK:
        return P.lib().ri_fock_jk(N, na, no, B, prec, p, p, n_pairs, p, p, p, None, p, nb, None)
    if op == Bd.OP_ENERGY:
        o, r = Bd.SCFOpts(10, 6, 1e-10, 1e-8, 0, 0), Bd.SCFResult()
        return P.lib().ri_energy(ctypes.byref(s), B, prec, p, p, n_pairs, ctypes.byref(o), None, p, p, None,
                                 ctypes.byref(r), p, nb, None)
    return P.lib().ri_gradient(ctypes.byref(s), p, n_pairs, B, prec, p, p, p, p, p, p, nb, None)


FORMS = [P.FP64, P.FP32, P.FP64 | P.COMPRESSED, P.FP32 | P.COMPRESSED, P.BF16X6]


@pytest.mark.parametrize("op,prec", [(op, prec) for op in (Bd.OP_FOCK, Bd.OP_ENERGY, Bd.OP_GRADIENT) for prec in FORMS]
                         + [(Bd.OP_ENERGY, P.FP32 | P.FINAL_FP64), (Bd.OP_ENERGY, P.BF16X6 | P.FINAL_FP64)])
def test_longer_list_covers_shorter(op, prec):
    torch = pytest.importorskip("torch")
    if torch.cuda.is_available():
        pytest.skip("runs on a host without a GPU")
    for N, na, no in ((40, 100, 4), (400, 1200, 40), (1000, 3000, 100)):
        full = N * (N + 1) // 2
        lists = [0, 1, full // 8, full * 3 // 5, full * 2 // 3, full]
        size = {n: Bd.workspace_bytes(op, N, na, no, n, prec) for n in lists}
        for longer in lists:
            for n in lists:
                if n <= longer:
                    assert _call(op, N, na, no, n, prec, size[longer]) == HIP, (N, longer, n)
        assert _call(op, N, na, no, full, prec, size[full] - 1) == WORKSPACE


@pytest.mark.parametrize("op", [Bd.OP_FOCK, Bd.OP_ENERGY, Bd.OP_GRADIENT])
@pytest.mark.parametrize("prec", [P.FP64, P.FP32])
def test_compressed_needs_no_slab_beside_the_lists(op, prec):
    torch = pytest.importorskip("torch")
    if torch.cuda.is_available():
        pytest.skip("runs on a host without a GPU")
    # X over the significant pairs: the size without the flag is enough
    for N, na, no, n in ((1000, 3000, 100, 68799), (440, 1320, 44, 24102)):
        nb = Bd.workspace_bytes(op, N, na, no, n, prec)
        assert nb < Bd.workspace_bytes(op, N, na, no, n, prec | P.COMPRESSED)
        assert _call(op, N, na, no, n, prec | P.COMPRESSED, nb) == HIP
    # a full list, and a small build: X slab by slab, which needs it
    for N, na, no, n in ((1000, 3000, 100, 500500), (40, 100, 4, 300)):
        nb = Bd.workspace_bytes(op, N, na, no, n, prec)
        assert _call(op, N, na, no, n, prec | P.COMPRESSED, nb) == WORKSPACE


def test_scf_holds_no_space_of_its_own_for_the_density_start():
    # the SCF's N x N matrices (13 and 16 of the DIIS ring), reduction scratch and N x n_occ blocks beside its Fock build,
    # and 256 MiB of room for the Fock build of a density start, which is over before the iterations begin
    for N, np_ in ((170, 11000), (400, 21000), (1000, 67325), (2000, 200000), (4000, 480000)):
        na, no = 3 * N, N // 10
        for prec in (P.FP64, P.FP32):
            extra = Bd.workspace_bytes(Bd.OP_ENERGY, N, na, no, np_, prec) - Bd.workspace_bytes(Bd.OP_FOCK, N, na, no, np_, prec)
            assert extra <= 30 * N * N * 8 + 6 * N * no * 8 + 4 * (N // 32 + 64) * 4096 * 8 + (256 << 20), (N, prec)
    # the build of a density itself: B^P and D B^P of a slab, at most 1 GiB each, the transposed copy of 64 auxiliaries
    for N, np_ in ((1000, 67325), (2000, 200000), (4000, 480000), (8000, 1200000)):
        nb = Bd.workspace_bytes(Bd.OP_FOCK_DENSITY, N, 3 * N, 1, np_, P.FP64)
        pad = (N + 127) // 128 * 128
        one = max(1 << 30, 8 * N * pad * 8)
        assert nb <= 2 * one + np_ * (64 + 17) * 8 + 4 * pad * pad * 8 + (N * (N + 256) * 8 + (1 << 25)), N


@pytest.mark.parametrize("prec", [P.FP64, P.FP32, P.FP32 | P.FINAL_FP64])
def test_batch_longer_lists_cover_shorter(prec):
    torch = pytest.importorskip("torch")
    if torch.cuda.is_available():
        pytest.skip("runs on a host without a GPU")
    d = ctypes.create_string_buffer(1 << 12)
    a = ctypes.cast(d, ctypes.c_void_p).value
    sizes = [(100, 300, 10), (149, 450, 14), (150, 450, 15), (333, 999, 33), (600, 1800, 60)]
    n = len(sizes)
    sys_ = (Bd.RISystem * n)(*[Bd.RISystem(N // 10, N, na, no, a, a, a, a, a, a) for N, na, no in sizes])

    def mols(f):
        return (Bd.BatchMol * n)(*[Bd.BatchMol(a, a, a, int(f * N * (N + 1) / 2), a, None) for N, _, _ in sizes])

    fills = [0.0, 0.01, 0.3, 0.59, 0.6, 0.61, 1.0]
    need = [P.lib().ri_energy_batched_workspace(n, ctypes.byref(sys_), ctypes.byref(mols(f)), prec) for f in fills]
    assert need == sorted(need)
    opts, res = Bd.SCFOpts(10, 6, 1e-10, 1e-8, 0, 0), (Bd.SCFResult * n)()
    for f, nb in zip(fills, need):
        args = [n, ctypes.byref(sys_), ctypes.byref(mols(f)), prec, ctypes.byref(opts), 0, None, ctypes.byref(res),
                ctypes.c_void_p(a)]
        assert P.lib().ri_energy_batched(*args, nb - 1, None) == WORKSPACE
        assert P.lib().ri_energy_batched(*args, need[-1], None) == HIP


@pytest.mark.parametrize("prec", [P.FP64, P.FP32])
def test_single_builds_of_dense_lists_stay_on_tiles(prec):
    # the copy of B_c for the partner lists is in the size where that form runs: one build with half of the pairs
    # significant is faster on resident tiles (and in FP64 the compressed form gives the same bits), the SCF over the lists
    W, size = Bd.workspace_bytes, 8 if prec == P.FP64 else 4
    for N in (400, 450, 500):
        na, no, half, few = 3 * N, N // 10, N * N // 4, N * N // 8
        copy = na * half * size
        jparts = 17 * 8 * (half + 1)
        full = N * (N + 1) // 2
        dense = W(Bd.OP_FOCK, N, na, no, full, prec)
        assert W(Bd.OP_FOCK, N, na, no, half, prec) <= dense
        assert W(Bd.OP_FOCK, N, na, no, few, prec) > dense - 17 * 8 * full + na * few * size
        comp = W(Bd.OP_FOCK, N, na, no, half, prec | P.COMPRESSED) - W(Bd.OP_FOCK, N, na, no, half, prec)
        assert comp < copy if prec == P.FP64 else comp > copy
        assert W(Bd.OP_ENERGY, N, na, no, half, prec) > W(Bd.OP_ENERGY, N, na, no, full, prec) - (256 << 20) - 17 * 8 * full + copy - jparts
