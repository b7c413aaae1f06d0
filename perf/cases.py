"""Performance cases of the spin-charge Krylov kernel: the calls that a program makes, over their range.

Every case is a dict of plain values; ``prepare`` builds the caller's inputs on the GPU from a
seed, ``run`` makes one pass through the public entry points, ``exact`` gives the same outputs from
plain torch operations in 64 bits and ``work`` the bytes and operations that a pass needs.

Kinds of case
  apply      K delta of rank m on a prepared handle: the call inside every solver iteration
  md_step    the electronic part of one extended-Lagrangian MD step: kk_prepare at the new
             eigenpairs, the ground-state charges, the adaptive-rank kernel on their residual and
             the update of the propagated charges
  response   density_response_batch: many first-order responses at one expansion point
  gradient   K delta and the reverse pass of L = |K delta|^2 (with or without the expansion
             point's Hamiltonians)
  batch      one update of many uneven clusters (krylov_kernel_apply_batch)
  mulliken   Mulliken sums of caller density-matrix changes

Systems are bcc iron as in the synthetic generator of this repository: a = 2.87 A, sites displaced
by 0.05 A, 9 orbitals an atom (with ``ragged``, 4 on about every third), overlaps that decay with
0.6 A within 5 A, S = I + 0.15 X / rho(X), the screened Coulomb matrix with U = 0.4 Ha,
W = -0.015 Ha, kT = 0.25 eV, 8 electrons for 9 orbitals. 2 c^3 atoms are a periodic cell, any other
count an open cluster. The eigenpairs are drawn, not solved for, so that inputs are quick to make at
every size: orthonormal Q with entries like those of delocalized states, and levels that follow the
generator's spectrum (a semicircle of radius 30 eV about -4.3 eV, the two spins 1.8 eV apart), in
ascending order as an eigensolver returns them.
"""

from __future__ import annotations

import math

import numpy as np
import torch

from paper_2303_03529_amd import krylov

DEV = "cuda"
F64 = torch.float64
HARTREE_EV, BOHR_ANG = 27.211386, 0.52917721
LATTICE, CUTOFF, DECAY, R0 = 2.87, 5.0, 0.6, 2.48
HUBBARD_HA, STONER_EV, KT = 0.4, -0.015 * HARTREE_EV, 0.25
CENTRE_EV, RADIUS_EV, SPLIT_EV = -4.3, 30.0, 0.9
PRECISION = {"fp64": krylov.KK_FP64, "f16": krylov.KK_MIXED_F16, "bf16": krylov.KK_MIXED_BF16}
# the adaptive kernel's settings of the SCF driver, and a sixth-order dissipative Verlet step
M_MAX, RANK_TOL = 8, 0.1
KAPPA, ALPHA, DISSIPATION = 1.82, 0.018, (-6.0, 14.0, -8.0, -3.0, 4.0, -1.0)


def listed():
    return [
        # the method paper's own 16-atom cell: an MD step there is a chain of short launches
        dict(name="md_step_16_fp64", kind="md_step", atoms=16, precision="fp64"),
        # the smallest update: latency and launches
        dict(name="apply_16_fp64", kind="apply", atoms=16, precision="fp64", m=4),
        # an odd open cluster with a dense preconditioner, split transforms
        dict(name="apply_37_f16_k0", kind="apply", atoms=37, precision="f16", m=6, dense_k0=True),
        # an MD step of the ordinary 128-atom cell on the split transforms
        dict(name="md_step_128_f16", kind="md_step", atoms=128, precision="f16"),
        # the ordinary update
        dict(name="apply_128_fp64", kind="apply", atoms=128, precision="fp64", m=8),
        # ragged orbital counts, an odd size between two tile classes, the BF16 form
        dict(name="apply_171_bf16_ragged", kind="apply", atoms=171, precision="bf16", m=8, ragged=True),
        # columns of the Jacobian at one expansion point
        dict(name="response_250_fp64", kind="response", atoms=250, precision="fp64", batch=8),
        # a large cell on the split transforms
        dict(name="apply_432_f16", kind="apply", atoms=432, precision="f16", m=8),
        # the headline: the largest cell, FP64, rank 12
        dict(name="apply_1024_fp64", kind="apply", atoms=1024, precision="fp64", m=12),
        # training through the kernel: all gradients
        dict(name="gradient_128_fp64", kind="gradient", atoms=128, precision="fp64", m=8, want_h=True),
        # many uneven clusters at once
        dict(name="batch_24_fp64", kind="batch", systems=24, lo=16, hi=250, precision="fp64", m=6),
        # density-matrix changes that the caller holds
        dict(name="mulliken_432", kind="mulliken", atoms=432, precision="fp64", batch=2),
    ]


def draw(rng):
    def atoms(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["apply", "apply", "apply", "md_step", "md_step", "response", "gradient", "batch", "mulliken"])
    precision = rng.choice(["fp64", "fp64", "f16", "bf16"])
    if kind == "apply":
        n = atoms(8, 500)
        return dict(kind=kind, atoms=n, precision=precision, m=rng.randint(2, 12), ragged=rng.random() < 0.3,
                    dense_k0=rng.random() < 0.2)
    if kind == "md_step":
        return dict(kind=kind, atoms=atoms(8, 300), precision=precision, ragged=rng.random() < 0.3)
    if kind == "response":
        return dict(kind=kind, atoms=atoms(8, 300), precision=precision, batch=rng.randint(1, 12),
                    ragged=rng.random() < 0.3)
    if kind == "gradient":
        return dict(kind=kind, atoms=atoms(12, 200), precision="fp64", m=rng.randint(2, 8),
                    want_h=rng.random() < 0.7)
    if kind == "batch":
        lo = rng.randint(16, 60)
        return dict(kind=kind, systems=rng.randint(6, 32), lo=lo, hi=lo + rng.randint(20, 130),
                    precision=rng.choice(["fp64", "f16"]), m=rng.randint(3, 8))
    return dict(kind=kind, atoms=atoms(16, 432), precision="fp64", batch=rng.randint(1, 4), ragged=rng.random() < 0.3)


# ---------------------------------------------------------------------------------------------
# Inputs


def orbital_counts(case, n):
    """Orbitals of each atom: 9 (s, p, d), or 4 (s, p) on about every third atom of a ragged case."""
    k = np.arange(n)
    return np.where((k * 0.6180339887) % 1.0 < 0.3, 4, 9) if case.get("ragged") else np.full(n, 9)


def cluster_sizes(case):
    k = np.arange(case["systems"])
    return [int(case["lo"] + (case["hi"] - case["lo"]) * x) for x in (0.5 + k * 0.6180339887) % 1.0]


def sites(n):
    """Ideal sites of n atoms and the box edge: a periodic cell for n = 2 c^3, else the n sites of an
    8^3-cell lattice nearest its centre and no box."""
    c = round((n / 2) ** (1 / 3))
    cells, box = (c, LATTICE * c) if 2 * c ** 3 == n else (8, None)
    g = np.stack(np.meshgrid(*[np.arange(cells)] * 3, indexing="ij"), -1).reshape(-1, 1, 3)
    x = LATTICE * (g + np.array([[0.0] * 3, [0.5] * 3])[None]).reshape(-1, 3)
    if box is None:
        d2 = ((x - x.mean(0)) ** 2).sum(1)
        x = x[np.sort(np.lexsort((np.arange(len(x)), d2))[:n])]
    return x, box


def semicircle_levels(nb):
    """Level k of nb at the quantile (k + 1/2) / nb of the unit semicircle density."""
    t = np.linspace(0.0, math.pi, 20001)          # x = -cos t, cumulative (t - sin t cos t) / pi
    return -np.cos(np.interp((np.arange(nb) + 0.5) / nb, (t - np.sin(t) * np.cos(t)) / math.pi, t))


def orthonormal(nb, gen):
    """A dense orthonormal matrix: cosine transforms with random signs and a random row order."""
    k = torch.arange(nb, dtype=F64, device=DEV)
    dct = torch.cos(math.pi / nb * k[:, None] * (k[None, :] + 0.5)) * math.sqrt(2.0 / nb)
    dct[0] *= math.sqrt(0.5)
    sign = [torch.randint(0, 2, (nb,), device=DEV, generator=gen).to(F64) * 2 - 1 for _ in range(2)]
    order = torch.randperm(nb, device=DEV, generator=gen)
    return ((dct * sign[0][None, :])[order] @ (dct * sign[1][:, None])).contiguous()


def make_system(n, counts, gen):
    """What a caller hands to kk_prepare, and its propagated charges' reference."""
    nb = int(counts.sum())
    x, box = sites(n)
    pos = torch.as_tensor(x, device=DEV) + 0.05 * torch.randn(n, 3, dtype=F64, device=DEV, generator=gen)
    diff = pos[None] - pos[:, None]
    if box:
        diff -= box * torch.round(diff / box)
    shifts = [(a, b, c) for a in (-1, 0, 1) for b in (-1, 0, 1) for c in (-1, 0, 1)] if box else [(0, 0, 0)]
    weight, r2 = torch.zeros(n, n, dtype=F64, device=DEV), torch.full((n, n), math.inf, dtype=F64, device=DEV)
    for s in shifts:
        d2 = ((diff + (box or 0.0) * torch.tensor(s, dtype=F64, device=DEV)) ** 2).sum(-1)
        r2 = torch.minimum(r2, d2)
        weight += torch.where(d2 < CUTOFF ** 2, torch.exp(-(d2.sqrt() - R0) / DECAY), 0.0)
    weight.fill_diagonal_(0.0)
    atom = torch.repeat_interleave(torch.arange(n, device=DEV), torch.as_tensor(counts, device=DEV))
    S = torch.randn(nb, nb, dtype=F64, device=DEV, generator=gen)
    S = torch.triu(S) + torch.triu(S, 1).T
    S *= weight[atom][:, atom]
    v = torch.ones(nb, dtype=F64, device=DEV)
    rho = 0.0
    for _ in range(24):                             # spectral radius, a little below the true one
        v = S @ (v / v.norm())
        rho = v.norm()
    S *= 0.15 / torch.clamp(1.05 * rho, min=1e-30)
    S += torch.eye(nb, dtype=F64, device=DEV)
    Z = torch.eye(nb, dtype=F64, device=DEV)        # S^-1/2 by Newton's iteration
    for _ in range(6):
        Z = 1.5 * Z - 0.5 * (Z @ S) @ (Z @ Z)
        Z = 0.5 * (Z + Z.T)
    base = torch.as_tensor(semicircle_levels(nb), device=DEV)
    out = dict(S=S.contiguous(), Z=Z.contiguous())
    for name, sign in (("up", -1.0), ("dn", 1.0)):
        jitter = 0.3 / nb * (torch.rand(nb, dtype=F64, device=DEV, generator=gen) - 0.5)
        out["eps_" + name] = torch.sort(CENTRE_EV + sign * SPLIT_EV + RADIUS_EV * (base + jitter)).values.contiguous()
        out["Q_" + name] = orthonormal(nb, gen)
    gamma = HARTREE_EV / torch.sqrt(r2 / BOHR_ANG ** 2 + 1.0 / HUBBARD_HA ** 2)
    gamma.fill_diagonal_(HUBBARD_HA * HARTREE_EV)
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    out.update(offsets=offsets, gamma=gamma.contiguous(), W=STONER_EV, kT=KT, n_electrons=8.0 * nb / 9.0)
    return out


def inputs(case, seed):
    gen = torch.Generator(device=DEV).manual_seed(int(seed))

    def randn(*shape, scale=1.0):
        return (torch.randn(*shape, dtype=F64, device=DEV, generator=gen) * scale).contiguous()

    if case["kind"] == "batch":
        s = dict(systems=[], delta=[])
        for n in cluster_sizes(case):
            s["systems"].append(make_system(n, orbital_counts(case, n), gen))
            s["delta"].append(randn(2 * n, scale=0.01))
        return s
    n = case["atoms"]
    counts = orbital_counts(case, n)
    s = dict(system=make_system(n, counts, gen), atoms=n)
    if case["kind"] in ("apply", "gradient"):
        s["delta"] = randn(2 * n, scale=0.01)
        if case.get("dense_k0"):                    # -I and a few percent of everything else
            s["K0"] = (-torch.eye(2 * n, dtype=F64, device=DEV) + randn(2 * n, 2 * n, scale=0.05 / math.sqrt(2 * n)))
    elif case["kind"] == "md_step":
        s["valence"] = torch.as_tensor(8.0 / 9.0 * counts, dtype=F64, device=DEV).contiguous()
        n_now = charges(Reference(s["system"]), s["valence"]) + randn(2 * n, scale=0.01)
        s["hist"] = (n_now[None] + randn(len(DISSIPATION), 2 * n, scale=0.001)).contiguous()
        s["c"] = torch.tensor(DISSIPATION, dtype=F64, device=DEV)
    elif case["kind"] == "response":
        s["v"] = randn(case["batch"], 2 * n)
    elif case["kind"] == "mulliken":
        nb = int(counts.sum())
        s["dD"] = []
        for _ in range(2):
            d = randn(case["batch"], nb, nb, scale=1e-3)
            s["dD"].append((d + d.transpose(1, 2)).contiguous())
    return s


def prepare_handle(handle, y, precision):
    handle.prepare(y["offsets"], y["S"], y["Z"], y["Q_up"], y["Q_dn"], y["eps_up"], y["eps_dn"], y["gamma"], y["W"],
                   y["kT"], y["n_electrons"], precision)


def prepare(case, seed):
    s = inputs(case, seed)
    s["case"], s["precision"] = case, PRECISION[case["precision"]]
    if case["kind"] == "batch":
        # the tile classes and workgroups per CU that the autotuner finds for such a batch
        s["batch"] = krylov.Batch().prepare(s.pop("systems"), s["precision"]).set_tuning(512, 4)
        s["outs"] = [torch.empty_like(d) for d in s["delta"]]
        return s
    s["handle"] = krylov.Handle()
    if case["kind"] != "md_step":                   # an MD step prepares its own expansion point
        prepare_handle(s["handle"], s.pop("system"), s["precision"])
    if "delta" in s:
        s["out"] = torch.empty_like(s["delta"])
    return s


def run(s):
    case, kind = s["case"], s["case"]["kind"]
    if kind == "batch":
        return s["batch"].krylov_kernel_apply(s["delta"], case["m"], s["outs"], info=False)[0]
    h = s["handle"]
    if kind == "apply":
        return h.krylov_kernel_apply(s["delta"], case["m"], K0=s.get("K0"), out=s["out"], info=False)[0]
    if kind == "response":
        return h.density_response_batch(s["v"])
    if kind == "mulliken":
        return h.mulliken_project(*s["dD"])
    if kind == "gradient":
        x = h.krylov_kernel_apply(s["delta"], case["m"], out=s["out"], info=False)[0]
        g = h.krylov_kernel_adjoint(s["delta"], case["m"], 2.0 * x, reuse_forward=True, want_H=case["want_h"])
        return dict(x=x, delta=g["delta"], gamma=g["gamma"], W=g["W"], H_up=g["H_up"], H_dn=g["H_dn"])
    prepare_handle(h, s["system"], s["precision"])
    q = h.ground_state_charges(s["valence"])
    f = q - s["hist"][0]
    Kf, info = h.krylov_kernel_apply_adaptive(f, M_MAX, RANK_TOL)
    n_new = h.xlbomd_update(s["hist"], Kf, KAPPA, ALPHA, s["c"])
    return dict(q=q, Kf=Kf, n_new=n_new, rank=info.rank_used)


# ---------------------------------------------------------------------------------------------
# The same in plain torch, 64 bits


def fermi_divided_differences(eps, mu):
    """(f_i - f_j) / (e_i - e_j) and f' on the diagonal, without cancellation."""
    lo, hi = torch.minimum(eps[:, None], eps[None]), torch.maximum(eps[:, None], eps[None])
    z = (lo - hi) / KT
    close = z == 0.0
    phi = torch.where(close, 1.0, torch.expm1(z) / torch.where(close, 1.0, z))
    return -torch.sigmoid((mu - lo) / KT) * torch.sigmoid((hi - mu) / KT) * phi / KT


class Reference:
    """Responses at one expansion point; eps and C may carry gradients."""

    def __init__(self, y, eps=None, C=None, gamma=None, W=None):
        self.n = len(y["offsets"]) - 1
        self.atom = torch.repeat_interleave(torch.arange(self.n, device=DEV),
                                            torch.as_tensor(np.diff(y["offsets"]), device=DEV))
        self.gamma, self.W = y["gamma"] if gamma is None else gamma, y["W"] if W is None else W
        self.eps = eps or [y["eps_up"], y["eps_dn"]]
        self.C = C or [y["Z"] @ y["Q_up"], y["Z"] @ y["Q_dn"]]
        self.G = [y["S"] @ c for c in self.C]
        e = torch.cat([x.detach() for x in self.eps])
        lo, hi = float(e.min()) - 40 * KT, float(e.max()) + 40 * KT
        for _ in range(70):
            mid = 0.5 * (lo + hi)
            lo, hi = (mid, hi) if float(torch.sigmoid((mid - e) / KT).sum()) < y["n_electrons"] else (lo, mid)
        mu = 0.5 * (lo + hi)
        for _ in range(2):   # Newton; through the last step the levels' gradients reach mu
            mu = float(mu)
            both = torch.cat(list(self.eps))
            f = torch.sigmoid((mu - both) / KT)
            w = (f * torch.sigmoid((both - mu) / KT)).detach() / KT
            mu = mu + (y["n_electrons"] - f.sum()) / w.sum()
        self.mu = mu
        self.f = [torch.sigmoid((mu - x) / KT) for x in self.eps]
        self.w = [f * torch.sigmoid((x - mu) / KT) / KT for f, x in zip(self.f, self.eps)]
        self.F = [fermi_divided_differences(x, mu) for x in self.eps]

    def atoms(self, rows):
        return torch.zeros(self.n, dtype=F64, device=DEV).index_add(0, self.atom, rows)

    def response(self, v):
        n = self.n
        X, top = [], 0.0
        for s, sign in enumerate((1.0, -1.0)):
            u = (self.gamma @ v[:n] + sign * self.W * v[n:])[self.atom]
            A = self.C[s].T @ (u[:, None] * self.G[s])
            X.append(0.5 * (A + A.T))
            top = top + (self.w[s] * X[s].diagonal()).sum()
        dmu = top / (self.w[0].sum() + self.w[1].sum())
        d = [self.atoms(((self.C[s] @ (self.F[s] * X[s] + torch.diag(dmu * self.w[s]))) * self.G[s]).sum(1))
             for s in (0, 1)]
        return torch.cat([d[0] + d[1], d[0] - d[1]])

    def kernel(self, delta, m, K0=None, tol=0.0):
        pre = (lambda x: -x) if K0 is None else (lambda x: K0 @ x)
        ft = pre(delta)
        V, Fs, r = [], [], ft
        for _ in range(m):
            for _ in range(2):
                for v in V:
                    r = r - (v @ r) * v
            V.append(r / r.norm())
            Fs.append(pre(self.response(V[-1]) - V[-1]))
            r = Fs[-1]
            F = torch.stack(Fs, 1)
            c = torch.linalg.solve(F.T @ F, F.T @ ft)
            if tol > 0.0 and float((F @ c - ft).norm()) <= tol * float(ft.norm()):
                break
        return torch.stack(V, 1) @ c, len(V)


def charges(ref, valence):
    p = [ref.atoms((ref.C[s] * ref.G[s] * ref.f[s]).sum(1)) for s in (0, 1)]
    return torch.cat([p[0] + p[1] - valence, p[0] - p[1]])


def exact(case, seed):
    s = inputs(case, seed)
    kind, m = case["kind"], case.get("m")
    if kind == "batch":
        return [Reference(y).kernel(d, m)[0] for y, d in zip(s["systems"], s["delta"])]
    y, n = s["system"], s["atoms"]
    if kind == "mulliken":
        atom = Reference(y).atom
        rows = [[torch.zeros(n, dtype=F64, device=DEV).index_add(0, atom, (d * y["S"]).sum(1)) for d in ds]
                for ds in s["dD"]]
        return torch.stack([torch.cat([a + b, a - b]) for a, b in zip(*rows)])
    if kind == "gradient":
        return exact_gradient(case, y, s["delta"])
    ref = Reference(y)
    if kind == "apply":
        return ref.kernel(s["delta"], m, s.get("K0"))[0]
    if kind == "response":
        return torch.stack([ref.response(v) for v in s["v"]])
    q = charges(ref, s["valence"])
    Kf, rank = ref.kernel(q - s["hist"][0], M_MAX, tol=RANK_TOL)
    n_new = 2 * s["hist"][0] - s["hist"][1] - KAPPA * Kf + ALPHA * (s["c"][:, None] * s["hist"]).sum(0)
    return dict(q=q, Kf=Kf, n_new=n_new, rank=rank)


def exact_gradient(case, y, delta):
    """torch.autograd through the levels, the eigenvectors and mu. gamma and W enter through the
    response potentials only, as in the library's reverse pass."""
    delta, gamma = delta.clone().requires_grad_(), y["gamma"].clone().requires_grad_()
    W = torch.tensor(y["W"], dtype=F64, device=DEV, requires_grad=True)
    wanted, eps, C = [delta, gamma, W], None, None
    if case["want_h"]:
        eps, C = [], []
        for spin in ("up", "dn"):
            B = y["S"] @ (y["Z"] @ y["Q_" + spin])
            H = ((B * y["eps_" + spin]) @ B.T).requires_grad_()
            P = y["Z"].T @ H @ y["Z"]
            e, Q = torch.linalg.eigh(0.5 * (P + P.T))
            eps.append(e)
            C.append(y["Z"] @ Q)
            wanted.append(H)
    x = Reference(y, eps, C, gamma, W).kernel(delta, case["m"])[0]
    g = torch.autograd.grad((x * x).sum(), wanted)
    H = [0.5 * (h + h.T) for h in g[3:]] or [None, None]
    return dict(x=x.detach(), delta=g[0], gamma=g[1], W=g[2], H_up=H[0], H_dn=H[1])


# ---------------------------------------------------------------------------------------------
# What a pass cannot do without


def work(case):
    """Each input read once and each output written once; two products of 2 Nb^3 operations per
    spin and direction."""
    m = case.get("m", 0)
    if case["kind"] == "batch":
        each = [work(dict(case, kind="apply", atoms=n)) for n in cluster_sizes(case)]
        return {k: sum(w[k] for w in each) for k in ("bytes", "flops")}
    n = case["atoms"]
    nb = int(orbital_counts(case, n).sum())
    matrices = 8.0 * nb * nb
    if case["kind"] == "apply":      # C and G of both spins; two vectors; K0
        return dict(bytes=4 * matrices + 32.0 * n + (32.0 * n * n if case.get("dense_k0") else 0.0),
                    flops=8.0 * m * nb ** 3)
    if case["kind"] == "response":
        return dict(bytes=4 * matrices + 32.0 * n * case["batch"], flops=8.0 * case["batch"] * nb ** 3)
    if case["kind"] == "mulliken":   # dD of both spins and S
        return dict(bytes=(2 * case["batch"] + 1) * matrices + 16.0 * n * case["batch"],
                    flops=4.0 * case["batch"] * nb * nb)
    if case["kind"] == "gradient":   # forward, transposed responses; X and Y of v_k and the commutators for H
        return dict(bytes=(6 if case["want_h"] else 4) * matrices + 8.0 * n * n,
                    flops=(28.0 * m + 8.0 if case["want_h"] else 16.0 * m) * nb ** 3)
    # md_step: C = Z Q and G = S C of both spins, then at least one direction
    return dict(bytes=4 * matrices + 8.0 * n * n, flops=16.0 * nb ** 3)
