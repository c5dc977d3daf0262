"""The calls a user of this framework makes, with their sizes, as cases that can be timed and checked.

Systems are the repository's synthetic ones: helium-like centres drawn in a ball at 0.01 per
cubic bohr with 10 orbital and 30 auxiliary functions each (N = 100 to 1000, the range of the
benchmark's workloads), and the 8-centre cube with 4 and 10 functions each (N = 32).  Every
size follows from the number of centres, which goes through odd values as well as the
benchmark's 40 and 100; geometries come from the seed.

    scf       ri_energy from the core Hamiltonian, or from the orbitals of a displaced geometry
              (the start of a dynamics step)
    fock      one J/K build from occupied orbitals: FP64, FP32 or split-BF16 exchange
    density   one J/K build from a density matrix (a predicted density as a start)
    setup     a new geometry up to its first J and K: pairs, three-centre integrals, metric factor,
              B, and one build from orbitals in hand
    gradient  nuclear gradient at converged orbitals (the backward direction of every dynamics step)
    batch     lockstep SCF of many molecules, with the tuned launch shapes
    features  pair features and the learned start's network on them
    train     one training step of that network

The metric's condition number reaches 1e14, so the fitted tensor B, its factor and gamma are
determined to about 1e-9 only, and orbitals only up to a rotation: what is compared is what they
stand for, J, K, F, D, energies and gradients.
"""
import math
import types

import numpy as np
import torch

from paper_2407_19614_amd import binding, learned

PREC = {"fp64": binding.FP64, "fp32": binding.FP32, "bf16x3": binding.BF16X3, "bf16x6": binding.BF16X6}
STORED = {"fp64": 8, "fp32": 4, "bf16x3": 4, "bf16x6": 6}     # bytes of an element of B
FIN = binding.FP32 | binding.FINAL_FP64
TRAIN_STEP, TRAIN_LR = 500, 1e-3


# ---------------------------------------------------------------- cases
def listed():
    return [
        # smallest whole call: the 8-centre system of the smoke test, all launches and host waits
        {"name": "scf-8", "op": "scf", "centres": 8, "start": "core"},
        # a step of the 40-centre geometry sequence, from the previous geometry's orbitals
        {"name": "scf-40-next", "op": "scf", "centres": 40, "start": "previous"},
        # the first SCF of a molecule of no special size
        {"name": "scf-27", "op": "scf", "centres": 27, "start": "core"},
        # the benchmark's Fock build, N = 1000
        {"name": "fock-100", "op": "fock", "centres": 100, "prec": "fp64"},
        # an ordinary molecule, no dimension a multiple of a tile
        {"name": "fock-37", "op": "fock", "centres": 37, "prec": "fp64"},
        # reduced-precision exchange at FP32-like accuracy, a size between the benchmark's
        {"name": "fock-73-bf16x6", "op": "fock", "centres": 73, "prec": "bf16x6"},
        # a new geometry of the largest workload, and of a small molecule
        {"name": "setup-100", "op": "setup", "centres": 100, "prec": "fp64"},
        {"name": "setup-17", "op": "setup", "centres": 17, "prec": "fp64"},
        # forces of the largest workload (a dynamics step)
        {"name": "gradient-100", "op": "gradient", "centres": 100},
        # many molecules at once: FP32 iterations and a final FP64 exchange build, as the benchmark runs them
        {"name": "batch-60", "op": "batch", "molecules": 60, "low": 10, "high": 60, "prec": "fp32f64"},
        # the learned start on one geometry of the sequence, BF16 inference
        {"name": "features-40", "op": "features", "centres": 40, "prec": "bf16"},
        # one mini-batch of its training, FP32
        {"name": "train-16384", "op": "train", "rows": 16384},
    ]


def draw(rng):
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    op = rng.choice(["scf", "scf", "fock", "fock", "setup", "gradient", "batch", "density", "features", "train"])
    if op == "scf":
        return {"op": op, "centres": size(8, 100), "start": rng.choice(["core", "previous"])}
    if op == "fock":
        return {"op": op, "centres": size(8, 100), "prec": rng.choice(["fp64", "fp64", "fp32", "bf16x3", "bf16x6"])}
    if op == "setup":
        return {"op": op, "centres": size(8, 100), "prec": rng.choice(["fp64", "fp32", "bf16x6"])}
    if op == "gradient":
        return {"op": op, "centres": size(8, 100)}
    if op == "density":
        return {"op": op, "centres": size(10, 80)}
    if op == "batch":
        low = rng.randint(8, 24)
        return {"op": op, "molecules": size(4, 48), "low": low, "high": low + rng.randint(4, 24),
                "prec": rng.choice(["fp64", "fp32f64"])}
    if op == "features":
        return {"op": op, "centres": size(8, 100), "prec": rng.choice(["bf16", "fp32"])}
    return {"op": op, "rows": size(500, 32768)}


# ---------------------------------------------------------------- inputs
def cluster(n, rng):
    """n points at least 2.5 bohr apart: in a 10-bohr cube (8 or 9 of them), else in a ball at 0.01 per cubic bohr."""
    cube = n < 10
    r = 5.0 if cube else (3.0 * n / (4.0 * math.pi * 0.01)) ** (1.0 / 3.0)
    pts = np.zeros((0, 3))
    while len(pts) < n:
        p = rng.uniform(-r, r, size=3)
        if (cube or p @ p <= r * r) and (len(pts) == 0 or ((pts - p) ** 2).sum(1).min() >= 6.25):
            pts = np.vstack([pts, p])
    return pts


def system(n, rng):
    orb, aux, tau = (((0.3, 1.0, 3.5, 12.0), [0.1 * 2.5 ** k for k in range(10)], 0.0) if n < 10 else
                     ([0.08 * 2.2 ** k for k in range(10)], [0.05 * 1.6 ** k for k in range(30)], 1e-12))
    at = np.arange(n, dtype=np.int32)
    return types.SimpleNamespace(
        xyz=cluster(n, rng), Z=np.full(n, 2.0), fn_centre=np.tile(at, len(orb)), fn_exp=np.repeat(np.array(orb), n),
        aux_centre=np.tile(at, len(aux)), aux_exp=np.repeat(np.array(aux), n), n_centres=n, N=n * len(orb),
        n_aux=n * len(aux), n_occ=n, tau=tau)


def displaced(s, rng):
    return types.SimpleNamespace(**{**vars(s), "xyz": s.xyz + rng.normal(0.0, 0.05, s.xyz.shape)})


def orbitals(s, rng):
    return rng.standard_normal((s.N, s.n_occ)) / math.sqrt(s.N)


def density(s, rng):
    c = orbitals(s, rng)
    e = rng.standard_normal((s.N, s.N)) * (1e-3 / s.N)
    return 2.0 * c @ c.T + e + e.T


def molecules(case, rng):
    """Their sizes belong to the case, their geometries to the seed."""
    sizes = np.random.default_rng(case["molecules"]).integers(case["low"], case["high"] + 1, size=case["molecules"])
    return [system(int(n), rng) for n in sizes]


def turned(n, rng):
    """One cluster of n centres in another place, orientation and order: its number of pairs stays what it is."""
    s = system(n, np.random.default_rng(n))
    q, r = np.linalg.qr(rng.standard_normal((3, 3)))
    s.xyz = np.ascontiguousarray(rng.permutation(s.xyz @ (q * np.sign(np.diag(r))).T + rng.uniform(-1, 1, 3)))
    return s


def weights(rng):
    """A network in training: He-scaled weights with small biases."""
    w, nf = 256, 8
    parts = [rng.standard_normal(nf * w) * math.sqrt(2.0 / nf), rng.normal(0, 0.1, w),
             rng.standard_normal(w * w) * math.sqrt(2.0 / w), rng.normal(0, 0.1, w),
             rng.standard_normal(w) * math.sqrt(1.0 / w), rng.normal(0, 0.1, 1)]
    return np.concatenate(parts).astype(np.float32)


def training_rows(n, rng):
    """Features in the ranges that their normalisation assumes, and targets of a density's size."""
    f = np.empty((n, 8), np.float32)
    f[:, 0] = rng.uniform(0, 15, n)
    a, b = rng.uniform(-2.6, 4.6, n), rng.uniform(-2.6, 4.6, n)
    f[:, 1], f[:, 2] = np.maximum(a, b), np.minimum(a, b)
    f[:, 3] = rng.random(n) < 0.1
    f[:, 4] = np.exp(-0.3 * f[:, 0])
    c, d = rng.uniform(0, 3, n), rng.uniform(0, 3, n)
    f[:, 5], f[:, 6] = np.maximum(c, d), np.minimum(c, d)
    f[:, 7] = rng.uniform(0, 3, n)
    return f, (f[:, 4] * rng.standard_normal(n)).astype(np.float32)


def moments(rng):
    """Adam's moments some hundred steps into a training."""
    v = rng.uniform(0.5, 2.0, binding.NPARAM) * 1e-4
    return (rng.standard_normal(binding.NPARAM) * 1e-3).astype(np.float32), v.astype(np.float32)


def problem(s, prec=binding.FP64):
    pr = binding.RIProblem(s, device="cuda", prec=prec)
    pr.build_3c()
    pr.metric_factor(prec)
    return pr


def dev(a):
    return torch.tensor(np.ascontiguousarray(a), device="cuda")


def prepare(case, seed):
    rng = np.random.default_rng(seed)
    op = case["op"]
    st = {"op": op}
    if op == "batch":
        mols = molecules(case, rng)
        st["prec"] = FIN if case["prec"] == "fp32f64" else binding.FP64
        st["tol"] = dict(tol_E=1e-6, tol_err=3e-5) if case["prec"] == "fp32f64" else dict(tol_E=1e-10, tol_err=1e-8)
        st["prs"] = binding.prepare_batch(mols, prec=st["prec"])
        st["tuning"] = binding.BatchTuning()                      # the shapes that the tuner picks on this workload
        st["tuning"].n_buckets = binding.TUNE_BUCKETS
        for b in range(binding.TUNE_BUCKETS):
            st["tuning"].gemm_tile[b], st["tuning"].syrk_split[b] = 64, 16
        return st
    if op == "train":
        feat, target = training_rows(case["rows"], rng)
        st["net"] = binding.MLP(weights(rng), learned.FEAT_SHIFT, learned.FEAT_SCALE)
        m, v = moments(rng)
        st["net"].m.copy_(dev(m))
        st["net"].v.copy_(dev(v))
        st["net"].step = TRAIN_STEP
        st["feat"], st["target"] = dev(feat), dev(target)
        return st
    s = turned(case["centres"], rng) if op == "features" else system(case["centres"], rng)
    if op == "scf":
        st["guess"] = None
        if case["start"] == "previous":
            before = problem(displaced(s, rng))
            st["guess"] = before.energy()[1]
        st["pr"] = problem(s)
    elif op == "fock":
        st["pr"], st["C"] = problem(s, PREC[case["prec"]]), dev(orbitals(s, rng))
    elif op == "density":
        st["pr"], st["D"] = problem(s), dev(density(s, rng))
    elif op == "setup":
        st["pr"], st["C"] = binding.RIProblem(s, device="cuda", prec=PREC[case["prec"]]), dev(orbitals(s, rng))
    elif op == "gradient":
        st["pr"] = problem(s)
        _, st["C"], st["F"], _ = st["pr"].energy()
    elif op == "features":
        st["net"] = binding.MLP(weights(rng), learned.FEAT_SHIFT, learned.FEAT_SCALE)
        st["prec"] = binding.MLP_BF16 if case["prec"] == "bf16" else binding.MLP_FP32
        st["pr"] = binding.RIProblem(s, device="cuda")
        st["pr"].build_3c()
    return st


# ---------------------------------------------------------------- the calls
ENERGIES = ("E_total", "E_nuc", "E_1e", "E_J", "E_K")


def run(st):
    op = st["op"]
    if op == "scf":
        r, C, F, D = st["pr"].energy(guess=st["guess"])
        return {"E": np.array([r[k] for k in ENERGIES]), "F": F, "D": D}
    if op == "fock":
        J, K, _ = st["pr"].fock_jk(st["C"])
        return {"J": J, "K": K}
    if op == "density":
        J, K = st["pr"].fock_jk_density(st["D"])
        return {"J": J, "K": K}
    if op == "setup":
        pr = st["pr"]
        pr.build_3c()
        pr.metric_factor()
        J, K, _ = pr.fock_jk(st["C"])
        return {"J": J, "K": K}
    if op == "gradient":
        return st["pr"].gradient(st["C"], st["F"])
    if op == "batch":
        res, _, F = binding.energy_batched(st["prs"], prec=st["prec"], tuning=st["tuning"], want_fock=True, **st["tol"])
        return {"E": np.array([[r[k] for k in ENERGIES] for r in res]), "F": F}
    if op == "features":
        feat = st["pr"].pair_features()
        return {"feat": feat, "y": st["net"].forward(feat, st["prec"])}
    net = st["net"]
    loss, grad = net.train_step(st["feat"], st["target"], TRAIN_LR, want_grad=True)
    return {"loss": loss, "grad": grad, "params": net.params, "m": net.m, "v": net.v}


# ---------------------------------------------------------------- what a pass cannot do without
def n_pairs(s):
    d2 = ((s.xyz[:, None] - s.xyz[None]) ** 2).sum(-1)[s.fn_centre][:, s.fn_centre]
    a, b = s.fn_exp[:, None], s.fn_exp[None]
    p = a + b
    q = ((4.0 * a * b / math.pi ** 2) ** 0.75 * np.exp(-a * b / p * d2)) ** 2 * 2.0 * math.pi ** 2.5 / (p * p * np.sqrt(2.0 * p))
    return int(np.tril(q > s.tau).sum())


def fock_work(s, np_, stored=8):
    N, A, o = s.N, s.n_aux, s.n_occ
    # X = B C (all rows), the lower triangle of K, gamma and J on the pairs
    return {"bytes": stored * A * N * (N + 1) / 2 + 8.0 * A * np_ + 8 * N * (o + 2 * N),
            "flops": 2.0 * N * N * o * A + 1.0 * N * (N + 1) * o * A + 4.0 * A * np_}


def scf_work(s, np_, builds, stored=8):
    # one Fock build and about 30 symmetric squares (purification) and 4 products of N x N a step
    f = fock_work(s, np_, stored)
    return {"bytes": builds * f["bytes"], "flops": builds * (f["flops"] + 38.0 * s.N ** 3)}


def work(case):
    rng = np.random.default_rng(0)
    op = case["op"]
    if op == "batch":
        each = [scf_work(s, n_pairs(s), 12 if case["prec"] == "fp64" else 9, 8 if case["prec"] == "fp64" else 4)
                for s in molecules(case, rng)]
        return {k: sum(w[k] for w in each) for k in ("bytes", "flops")}
    if op == "train":
        n, p = case["rows"], 8 * 256 + 256 * 256 + 256
        return {"bytes": 4.0 * (9 * n + 7 * p), "flops": 6.0 * n * p - 2.0 * n * 8 * 256}
    s = system(case["centres"], rng)
    np_ = n_pairs(s)
    N, A, o = s.N, s.n_aux, s.n_occ
    if op == "scf":
        return scf_work(s, np_, 7 if case["start"] == "previous" else 13)
    if op == "fock":
        return fock_work(s, np_, STORED[case["prec"]])
    if op == "density":
        return {"bytes": 8.0 * A * np_ + 24.0 * N * N, "flops": 3.0 * N ** 3 * A + 4.0 * A * np_}
    if op == "setup":
        # about 40 operations an integral; Cholesky, the solve for B on the pairs, the factor's inverse; one build
        f = fock_work(s, np_, STORED[case["prec"]])
        return {"bytes": f["bytes"] + 8.0 * A * np_ + STORED[case["prec"]] * A * N * (N + 1) / 2 + 16.0 * A * A,
                "flops": f["flops"] + 40.0 * A * np_ + A ** 3 / 3 + 1.0 * A * A * np_ + A ** 3 / 3}
    if op == "gradient":
        # X and B_ij, Xi, its square, U, the products at the pairs, about 80 operations a derivative integral
        return {"bytes": 8.0 * A * N * (N + 1) / 2 + 8.0 * A * np_ + 8.0 * A * A,
                "flops": 2.0 * N * N * o * A + 2.0 * N * o * o * A + 1.0 * A * A * o * o + 1.0 * A * A * o * o
                + 2.0 * N * o * o * A + 2.0 * np_ * o * A + 80.0 * np_ * A}
    return {"bytes": np_ * (8.0 + 32 + 4) + 4.0 * binding.NPARAM,
            "flops": np_ * (2.0 * (8 * 256 + 256 * 256 + 256) + 30.0 * s.n_centres)}


# ---------------------------------------------------------------- the same in 64 bits, by plain torch
def boys(t):
    """F0(t), differentiable: its Taylor series below 1, erf above."""
    small = t < 1.0
    u = torch.where(small, t, torch.zeros_like(t))
    f = torch.zeros_like(t)
    for k in range(20, -1, -1):
        f = f * u + (-1.0) ** k / (math.factorial(k) * (2 * k + 1))
    r = torch.sqrt(torch.where(small, torch.ones_like(t), t))
    return torch.where(small, f, 0.5 * math.sqrt(math.pi) * torch.erf(r) / r)


def norm(a):
    return (2.0 * a / math.pi) ** 0.75


def solve(L, b, upper=False):
    return torch.linalg.solve_triangular(L.cpu(), b.cpu(), upper=upper).cuda()


class Plain:
    """Integrals, J/K and the SCF of one system in plain torch."""

    def __init__(self, s):
        self.s = s
        self.xyz = dev(s.xyz)
        self.fc, self.ac = dev(s.fn_centre).long(), dev(s.aux_centre).long()
        self.fe, self.ae, self.Z = dev(s.fn_exp), dev(s.aux_exp), dev(s.Z)
        d2 = ((self.xyz[:, None] - self.xyz[None]) ** 2).sum(-1)[self.fc][:, self.fc]
        p = self.fe[:, None] + self.fe[None]
        q = (norm(self.fe)[:, None] * norm(self.fe)[None] * torch.exp(-self.fe[:, None] * self.fe[None] / p * d2)) ** 2
        q = q * 2.0 * math.pi ** 2.5 / (p * p * torch.sqrt(2.0 * p))
        self.mu, self.nu = torch.nonzero(torch.tril(q > s.tau), as_tuple=True)
        self.w = torch.where(self.mu == self.nu, 1.0, 2.0).double()

    def gaussians(self, xyz, mu, nu):
        a, b = self.fe[mu], self.fe[nu]
        A, B = xyz[self.fc[mu]], xyz[self.fc[nu]]
        p = a + b
        r2 = ((A - B) ** 2).sum(-1)
        k = norm(a) * norm(b) * torch.exp(-a * b / p * r2)
        return p, (a[:, None] * A + b[:, None] * B) / p[:, None], k, a * b / p, r2

    def three_centre(self, xyz, lo, hi):
        p, P, k, _, _ = self.gaussians(xyz, self.mu, self.nu)
        c, C = self.ae[lo:hi, None], xyz[self.ac[lo:hi]]
        d2 = ((P[None] - C[:, None]) ** 2).sum(-1)
        return k * norm(c) * 2.0 * math.pi ** 2.5 / (p * c * torch.sqrt(p + c)) * boys(p * c / (p + c) * d2)

    def two_centre(self, xyz):
        a, b = self.ae[:, None], self.ae[None]
        d2 = ((xyz[:, None] - xyz[None]) ** 2).sum(-1)[self.ac][:, self.ac]
        return norm(a) * norm(b) * 2.0 * math.pi ** 2.5 / (a * b * torch.sqrt(a + b)) * boys(a * b / (a + b) * d2)

    def one_electron(self, xyz):
        """S and h over all pairs mu >= nu, as vectors, and the pairs."""
        m, n = torch.tril_indices(self.s.N, self.s.N, device="cuda")
        p, P, k, r, r2 = self.gaussians(xyz, m, n)
        S = k * (math.pi / p) ** 1.5
        h = S * r * (3.0 - 2.0 * r * r2)
        for c in range(self.s.n_centres):
            h = h - self.Z[c] * k * 2.0 * math.pi / p * boys(p * ((P - xyz[c]) ** 2).sum(-1))
        return m, n, S, h

    def nuclear(self, xyz):
        i, j = torch.triu_indices(self.s.n_centres, self.s.n_centres, 1, device="cuda")
        return (self.Z[i] * self.Z[j] / (xyz[i] - xyz[j]).norm(dim=-1)).sum()

    def dense(self, v, m, n):
        M = torch.zeros(v.shape[:-1] + (self.s.N, self.s.N), dtype=torch.float64, device="cuda")
        M[..., m, n] = v
        M[..., n, m] = v
        return M

    def factor(self):
        step = max(1, 30_000_000 // max(1, len(self.mu)))
        self.T = torch.cat([self.three_centre(self.xyz, k, min(k + step, self.s.n_aux)) for k in range(0, self.s.n_aux, step)])
        self.L = torch.linalg.cholesky(self.two_centre(self.xyz))
        self.Bc = solve(self.L, self.T)
        return self

    def slabs(self, n):
        step = max(1, 200_000_000 // (n * n))
        return [(k, min(k + step, self.s.n_aux)) for k in range(0, self.s.n_aux, step)]

    def jk(self, D, C=None):
        N = self.s.N
        J = self.dense((self.Bc @ (self.w * D[self.mu, self.nu])) @ self.Bc, self.mu, self.nu)
        K = torch.zeros_like(D)
        for lo, hi in self.slabs(N):
            B = self.dense(self.Bc[lo:hi], self.mu, self.nu).reshape(-1, N)
            X = (B @ (D if C is None else C)).reshape(hi - lo, N, -1).permute(1, 0, 2).reshape(N, -1)
            if C is None:
                K += 0.5 * X @ B
            else:
                K += X @ X.T
        return J, K

    def scf(self):
        N, o = self.s.N, self.s.n_occ
        m, n, S, h = self.one_electron(self.xyz)
        S, h, En = self.dense(S, m, n), self.dense(h, m, n), self.nuclear(self.xyz)
        X = solve(torch.linalg.cholesky(S), torch.eye(N, dtype=torch.float64, device="cuda"))
        F, fs, es = h, [], []
        for it in range(60):
            v = torch.linalg.eigh((X @ F @ X.T).cpu())[1].cuda()
            C = X.T @ v[:, :o]
            D = 2.0 * C @ C.T
            J, K = self.jk(D, C.contiguous())
            F = h + J - K
            M = F @ D @ S
            e = M - M.T
            parts = [(D * h).sum(), 0.5 * (D * J).sum(), -0.5 * (D * K).sum()]
            E = np.array([float(sum(parts) + En), float(En)] + [float(x) for x in parts])
            if float(e.abs().max()) < 2e-10:
                break
            fs, es = (fs + [F])[-7:], (es + [e])[-7:]
            G = torch.zeros(len(es) + 1, len(es) + 1, dtype=torch.float64)
            G[-1, :-1] = G[:-1, -1] = -1.0
            for i, a in enumerate(es):
                for j, b in enumerate(es):
                    G[i, j] = float((a * b).sum())
            G[:-1, :-1] /= G[:-1, :-1].abs().max()
            rhs = torch.zeros(len(es) + 1, dtype=torch.float64)
            rhs[-1] = -1.0
            c = torch.linalg.lstsq(G, rhs[:, None], driver="gelsd").solution[:, 0]
            Fx = sum(float(x) * f for x, f in zip(c, fs))
            F = Fx
        return E, C, h + J - K, D

    def gradient(self):
        """The derivative of the energy's terms with the density factors held, by automatic differentiation."""
        _, C, F, D = self.scf()
        s, N, A, o = self.s, self.s.N, self.s.n_aux, self.s.n_occ
        Bij = torch.empty((A, o * o), dtype=torch.float64, device="cuda")
        for lo, hi in self.slabs(N):
            X = (self.dense(self.Bc[lo:hi], self.mu, self.nu).reshape(-1, N) @ C).reshape(hi - lo, N, o)
            Bij[lo:hi] = (X.transpose(1, 2).reshape(-1, N) @ C).reshape(hi - lo, -1)
        gamma = self.Bc @ (self.w * D[self.mu, self.nu])
        both = solve(self.L.T, torch.cat([Bij, gamma[:, None]], 1), upper=True)
        Xi, c = both[:, :-1], both[:, -1].contiguous()
        Zm = c[:, None] * c[None] - 2.0 * Xi @ Xi.T
        W = 0.5 * D @ F @ D
        g = torch.zeros_like(self.xyz)

        def add(f):
            x = self.xyz.clone().requires_grad_(True)
            g.add_(torch.autograd.grad(f(x), x)[0])

        m, n = torch.tril_indices(N, N, device="cuda")
        w = torch.where(m == n, 1.0, 2.0).double()
        step = max(1, 100_000_000 // len(m)) if len(m) else 1
        Dv, Wv = w * D[m, n], w * W[m, n]
        for k in range(0, s.n_centres, step):                   # nuclear attraction by centres, to bound memory
            def attraction(x, k=k):
                p, P, q, _, _ = self.gaussians(x, m, n)
                e = sum(self.Z[i] * boys(p * ((P - x[i]) ** 2).sum(-1)) for i in range(k, min(k + step, s.n_centres)))
                return -(Dv * q * 2.0 * math.pi / p * e).sum()
            add(attraction)

        def overlap_kinetic(x):
            p, _, q, r, r2 = self.gaussians(x, m, n)
            S = q * (math.pi / p) ** 1.5
            return (Dv * S * r * (3.0 - 2.0 * r * r2)).sum() - (Wv * S).sum()
        add(overlap_kinetic)
        add(self.nuclear)
        add(lambda x: -0.5 * (Zm * self.two_centre(x)).sum())
        dm = D[self.mu, self.nu]
        step = max(1, min(100_000_000 // (N * N), 20_000_000 // max(1, len(self.mu))))
        for lo in range(0, A, step):
            hi = min(A, lo + step)
            U = (Xi[lo:hi].reshape(-1, o) @ C.T).reshape(hi - lo, o, N)     # Xi is symmetric in ij
            Y = torch.empty((hi - lo, len(self.mu)), dtype=torch.float64, device="cuda")
            for k in range(hi - lo):
                Y[k] = (C @ U[k])[self.mu, self.nu]
            Y = self.w * (c[lo:hi, None] * dm - 2.0 * Y)
            add(lambda x: (Y * self.three_centre(x, lo, hi)).sum())
        return g


def mlp(p, feat):
    """Pre-activations and outputs of the network in 64 bits."""
    v = torch.tensor(p, dtype=torch.float64, device="cuda")
    w1, b1, w2, b2, w3, b3 = torch.split(v, [8 * 256, 256, 256 * 256, 256, 256, 1])
    x = (feat - dev(learned.FEAT_SHIFT).double()) / dev(learned.FEAT_SCALE).double()
    leaves = [t.clone().requires_grad_(True) for t in (w1, b1, w2, b2, w3, b3)]
    w1, b1, w2, b2, w3, b3 = leaves
    h = torch.nn.functional.silu(x @ w1.view(8, 256) + b1)
    h = torch.nn.functional.silu(h @ w2.view(256, 256) + b2)
    return h @ w3 + b3, leaves


def exact(case, seed):
    rng = np.random.default_rng(seed)
    op = case["op"]
    if op == "batch":
        each = [Plain(s).factor().scf() for s in molecules(case, rng)]
        return {"E": np.array([e[0] for e in each]), "F": [e[2] for e in each]}
    if op == "train":
        feat, target = training_rows(case["rows"], rng)
        p = weights(rng)
        m, v = (dev(x).double() for x in moments(rng))
        y, leaves = mlp(p, dev(feat).double())
        loss = ((y - dev(target).double()) ** 2).mean()
        g = torch.cat(torch.autograd.grad(loss, leaves))
        k = TRAIN_STEP + 1
        m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
        new = torch.cat(leaves) - TRAIN_LR * (m / (1 - 0.9 ** k)) / (torch.sqrt(v / (1 - 0.999 ** k)) + 1e-8)
        return {"loss": loss.detach().reshape(1), "grad": g, "params": new.detach(), "m": m, "v": v}
    s = turned(case["centres"], rng) if op == "features" else system(case["centres"], rng)
    pl = Plain(s)
    if op == "features":
        p = weights(rng)
        r = pl.xyz
        near = torch.exp(-((r[:, None] - r[None]) ** 2).sum(-1) / 8.0).sum(1) - 1.0
        a, b = pl.fe[pl.mu], pl.fe[pl.nu]
        _, P, _, q, r2 = pl.gaussians(r, pl.mu, pl.nu)
        ca, cb = near[pl.fc[pl.mu]], near[pl.fc[pl.nu]]
        mid = torch.exp(-((P[:, None] - r[None]) ** 2).sum(-1) / 4.0).sum(1)
        feat = torch.stack([torch.sqrt(r2), torch.log(torch.maximum(a, b)), torch.log(torch.minimum(a, b)),
                            (pl.fc[pl.mu] == pl.fc[pl.nu]).double(), torch.exp(-q * r2), torch.maximum(ca, cb),
                            torch.minimum(ca, cb), mid], 1)
        return {"feat": feat, "y": mlp(p, feat)[0].detach()}
    if op == "gradient":
        return pl.factor().gradient()
    pl.factor()
    if op == "scf":
        E, _, F, D = pl.scf()
        return {"E": E, "F": F, "D": D}
    if op == "density":
        J, K = pl.jk(dev(density(s, rng)))
    else:
        C = dev(orbitals(s, rng))
        J, K = pl.jk(2.0 * C @ C.T, C)
    return {"J": J, "K": K}
