"""Performance cases of the central-eigenvalue library: what its users call, over the sizes they call it with.

Every case is a dict of plain values; its "op" names the entry point:

  apply          one y = H x on a block (the matrix-free step everything else is made of)
  estimates      the Lanczos bound and the Chebyshev density moments that set a window
  filter         the exp-semicircle filter of a start block
  basis          the evolution basis stored panel by panel
  stored         the same on the uniform grid, with S and P from the anchors' moments (the benchmark's way)
  moments        S and P from recorded moments, no basis stored
  project        S = V^T V and P = V^T (H V) of a stored basis
  ritz           the generalised eigenproblem of S and P, with its eigenvectors
  syev_batched   dense eigenproblems of many small subspaces in one call
  central        a whole call: the N levels nearest 0 of one Hamiltonian
  batch          a whole call over many disorder realisations

Hamiltonians are the chaotic Ising chain and the spin glass of the benchmark and the paper's own two models; their
couplings come from the seed.  Eigenvectors are returned with the sign that makes each one's largest component
positive, since an eigenvector's sign is free.  Whole calls return the levels; their error estimates are residuals at
the level of rounding and have no value of their own to compare.
"""
import math

import numpy as np
import torch

from paper_2011_02107_amd import binding as B
from paper_2011_02107_amd import inputs

DEV = "cuda:0"


# ------------------------------------------------------------------ cases

def listed():
    return [
        # one apply of a block of a small system: a launch and little else
        {"name": "apply_L14_b16", "op": "apply", "model": "chain", "L": 14, "b": 16, "dtype": "f64"},
        # the bound and density stage of a call, with the options' defaults
        {"name": "estimates_L16", "op": "estimates", "model": "chain", "L": 16, "steps": 80, "moments": 256, "nvec": 8},
        # the FP64 filter of a start block of the default width at a middle size
        {"name": "filter_L17_b64", "op": "filter", "model": "chain", "L": 17, "b": 64, "a_r": 0.06, "kfac": 18.0},
        # the evolution of a spin glass with a block width that fits no power of two
        {"name": "basis_L15_b23", "op": "basis", "model": "glass", "L": 15, "b": 23, "n": 7, "a_r": 0.02},
        # the benchmark's system size and its evolution with the moment projection, fewer samples and columns
        {"name": "stored_L20_b32", "op": "stored", "model": "chain", "L": 20, "b": 32, "n": 3, "a_r": 0.005},
        # a basis that is not kept: moments recorded along a longer evolution
        {"name": "moments_L16_b32", "op": "moments", "model": "chain", "L": 16, "b": 32, "n": 4, "a_r": 0.02},
        # the explicit projection of a stored basis, its width a multiple of nothing
        {"name": "project_L17_m1873", "op": "project", "model": "chain", "L": 17, "m": 1873},
        # the subspace problem of about 600 levels: S has the null space that an oversampled basis gives it
        {"name": "ritz_m1237", "op": "ritz", "m": 1237, "rank": 0.7},
        # the subspace problems of a round of small realisations
        {"name": "syev_batched_24", "op": "syev_batched", "count": 24, "n_lo": 90, "n_hi": 480},
        # the smallest whole call: the library's smoke size with its default options
        {"name": "central_L10_N100", "op": "central", "model": "chain", "L": 10, "N": 100, "b": 4, "tuned": False},
        # a whole call with the benchmark's options (FP32 filter with an FP64 tail, moment projection)
        {"name": "central_L16_N700_tuned", "op": "central", "model": "chain", "L": 16, "N": 700, "b": 64, "tuned": True},
        # the batched benchmark: 96 spin-glass realisations of three sizes
        {"name": "batch_96_N200", "op": "batch", "count": 96, "L_lo": 12, "L_hi": 14, "N": 200, "b": 16, "tuned": True},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["apply", "estimates", "filter", "basis", "stored", "moments", "project", "ritz", "syev_batched",
                     "central", "batch"])
    model = rng.choice(["chain", "chain", "glass", "tfim"])
    if op == "apply":
        return {"op": op, "model": rng.choice(["chain", "glass", "tfim", "sgs"]), "L": rng.randint(13, 19),
                "b": _log_int(rng, 4, 32), "dtype": rng.choice(["f64", "f32"])}
    if op == "estimates":
        return {"op": op, "model": model, "L": rng.randint(10, 18), "steps": rng.randint(40, 100),
                "moments": rng.randint(64, 256), "nvec": rng.randint(4, 8)}
    if op == "filter":
        return {"op": op, "model": model, "L": rng.randint(11, 18), "b": _log_int(rng, 2, 64),
                "a_r": round(math.exp(rng.uniform(math.log(0.04), math.log(0.3))), 4), "kfac": rng.choice([12.0, 18.0])}
    if op in ("basis", "stored"):
        return {"op": op, "model": model, "L": rng.randint(10, 19), "b": _log_int(rng, 2, 32), "n": rng.randint(2, 5),
                "a_r": round(math.exp(rng.uniform(math.log(0.01), math.log(0.1))), 4)}
    if op == "moments":
        return {"op": op, "model": model, "L": rng.randint(10, 16), "b": _log_int(rng, 2, 32), "n": rng.randint(2, 4),
                "a_r": round(math.exp(rng.uniform(math.log(0.02), math.log(0.1))), 4)}
    if op == "project":
        return {"op": op, "model": model, "L": rng.randint(11, 17), "m": _log_int(rng, 60, 1800)}
    if op == "ritz":
        return {"op": op, "m": _log_int(rng, 40, 1500), "rank": round(rng.uniform(0.5, 1.0), 2)}
    if op == "syev_batched":
        lo = _log_int(rng, 20, 200)
        return {"op": op, "count": rng.randint(2, 24), "n_lo": lo, "n_hi": lo + rng.randint(1, 280)}
    if op == "central":
        L = rng.randint(10, 16)
        return {"op": op, "model": rng.choice(["chain", "glass"]), "L": L,
                "N": _log_int(rng, 40, max(60, min(700, (1 << L) // 20))), "b": rng.choice([8, 16, 32]),
                "tuned": rng.choice([False, True])}
    lo = rng.randint(11, 13)
    return {"op": op, "count": rng.randint(4, 40), "L_lo": lo, "L_hi": rng.randint(lo, 14), "N": rng.randint(40, 100),
            "b": rng.choice([8, 16]), "tuned": rng.choice([False, True])}


# ------------------------------------------------------------------ inputs

def _terms(model, L, seed):
    if model == "chain":  # the benchmark's chaotic chain, its fields moved a little by the seed
        r = np.random.default_rng(seed)
        return inputs.ising_chain(L, hx=1.05 + 0.1 * r.uniform(), hz=0.5 + 0.1 * r.uniform())
    return {"glass": inputs.spin_glass, "tfim": inputs.paper_tfim, "sgs": inputs.paper_sgs}[model](L, seed)


def _bound(model, L, seed):
    """A bound above ||H|| such as the Lanczos estimate gives: the two-body and one-body parts' own sums where they
    can be had, else the sum of |c|."""
    t = _terms(model, L, seed)
    s = float(np.sqrt((t["coeff"] ** 2).sum()))
    return min(float(np.abs(t["coeff"]).sum()), 1.35 * s * math.sqrt(2.0 * L * math.log(2.0)))


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _block(D, b, seed, dtype=torch.float64):
    return torch.randn(D, b, generator=_gen(seed), device=DEV, dtype=torch.float64).to(dtype)


def _unit_block(D, b, seed):
    x = _block(D, b, seed)
    return (x / x.norm(dim=0)).contiguous()


def _goe(n, g):
    a = torch.randn(n, n, generator=g, device=DEV, dtype=torch.float64)
    return ((a + a.T) / math.sqrt(2.0 * n)).contiguous()


def _batched_sizes(case):
    c, lo, hi = case["count"], case["n_lo"], case["n_hi"]
    return [lo + (i * (hi - lo)) // max(1, c - 1) for i in range(c)]


def _pencil(case, seed):
    """S = C^T C' and P of an oversampled basis V = W C: rank r < m, a well conditioned range."""
    m = case["m"]
    r = max(1, min(m, int(round(case["rank"] * m))))
    g = _gen(seed)
    W = torch.randn(4 * r, r, generator=g, device=DEV, dtype=torch.float64) / math.sqrt(4.0 * r)
    lam = torch.rand(4 * r, generator=g, device=DEV, dtype=torch.float64) * 2 - 1
    C = torch.randn(r, m, generator=g, device=DEV, dtype=torch.float64) / math.sqrt(m)
    V = W @ C
    S = V.T @ V
    P = V.T @ (lam[:, None] * V)
    return (0.5 * (S + S.T)).contiguous(), (0.5 * (P + P.T)).contiguous(), r


def _opts(case, seed):
    if case["op"] == "batch":
        if case["tuned"]:  # the batched benchmark's tuned schedule
            return B.default_opts(b=case["b"], seed=seed, kfac=12.0, basis_ratio=1.3, precision=B.DACP_F32,
                                  fp64_tail_frac=0.3, moment_mode=2)
        return B.default_opts(b=case["b"], seed=seed)
    if case["tuned"]:
        return B.default_opts(b=case["b"], seed=seed, kfac=12.0, window_ratio=2.4, basis_ratio=1.2,
                              precision=B.DACP_F32, fp64_tail_frac=0.3, moment_mode=2)
    return B.default_opts(b=case["b"], seed=seed)


def _batch_sets(case, seed):
    span = case["L_hi"] - case["L_lo"] + 1
    return [(case["L_lo"] + i % span, inputs.spin_glass(case["L_lo"] + i % span, 1000 * (seed % 1000003) + i))
            for i in range(case["count"])]


def prepare(case, seed):
    s = {"case": case, "seed": seed, "ctx": B.Context(0)}
    op = case["op"]
    if op in ("ritz", "syev_batched"):
        if op == "ritz":
            s["S"], s["P"], s["r"] = _pencil(case, seed)
            s["B"] = torch.empty_like(s["S"])
        else:
            g = _gen(seed)
            s["A"] = [_goe(n, g) for n in _batched_sizes(case)]
            s["work"] = [torch.empty_like(a) for a in s["A"]]
            s["Z"] = [torch.empty_like(a) for a in s["A"]]
        return s
    if op == "batch":
        s["hams"] = [B.dacp_build_hamiltonian(s["ctx"], L, t) for L, t in _batch_sets(case, seed)]
        s["opts"] = _opts(case, seed)
        return s
    L = case["L"]
    D = 1 << L
    s["ham"] = B.dacp_build_hamiltonian(s["ctx"], L, _terms(case["model"], L, seed))
    if op == "apply":
        s["x"] = _block(D, case["b"], seed, torch.float32 if case["dtype"] == "f32" else torch.float64)
        s["y"] = torch.empty_like(s["x"])
    elif op == "estimates":
        s["v0"] = _block(D, 1, seed)
        s["R"] = _block(D, case["nvec"], seed + 1)
    elif op == "project":
        s["V"] = _block(D, case["m"], seed) / math.sqrt(D)
        s["S"] = torch.empty(case["m"], case["m"], device=DEV, dtype=torch.float64)
        s["P"] = torch.empty_like(s["S"])
    elif op == "central":
        s["opts"] = _opts(case, seed)
    else:
        s["e"] = _bound(case["model"], L, seed)
        s["a"] = case["a_r"] * s["e"]
        s["x"] = _unit_block(D, case["b"], seed)
        if op == "filter":
            s["K"] = _filter_order(case)
            s["y"] = torch.empty_like(s["x"])
        else:
            m = case["b"] * (2 * case["n"] + 1)
            if op != "moments":
                s["V"] = torch.empty(D, m, device=DEV, dtype=torch.float64)
            if op != "basis":
                s["S"] = torch.empty(m, m, device=DEV, dtype=torch.float64)
                s["P"] = torch.empty_like(s["S"])
    return s


# ------------------------------------------------------------------ one pass

def _signed(z):
    """Rows of eigenvectors with each one's largest component made positive."""
    big = z.gather(1, z.abs().argmax(dim=1, keepdim=True))
    return z * torch.where(big < 0, -1.0, 1.0)


def run(s):
    case, ctx = s["case"], s["ctx"]
    op = case["op"]
    if op == "apply":
        B.dacp_apply(ctx, s["ham"], s["x"], s["y"])
        return s["y"]
    if op == "estimates":
        e, lo, hi = B.dacp_spectral_bound(ctx, s["ham"], steps=case["steps"], v0=s["v0"])
        mu = B.dacp_dos_moments(ctx, s["ham"], e, case["moments"], nvec=case["nvec"], R=s["R"])
        return {"bound": np.array([e, lo, hi]), "mu": mu}
    if op == "filter":
        B.dacp_filter(ctx, s["ham"], s["y"], s["e"], s["a"], s["K"], start=s["x"])
        return s["y"]
    if op == "basis":
        B.dacp_basis(ctx, s["ham"], s["x"], s["V"], s["e"], s["a"], case["n"])
        return s["V"]
    if op == "stored":
        B.dacp_basis_stored_moments(ctx, s["ham"], s["x"], s["V"], s["S"], s["P"], s["e"], s["a"], case["n"])
        return {"V": s["V"], "S": s["S"], "P": s["P"]}
    if op == "moments":
        B.dacp_basis_moments(ctx, s["ham"], s["x"], s["S"], s["P"], s["e"], s["a"], case["n"])
        return {"S": s["S"], "P": s["P"]}
    if op == "project":
        B.dacp_project(ctx, s["ham"], s["V"], s["S"], s["P"])
        return {"S": s["S"], "P": s["P"]}
    if op == "ritz":
        theta, r = B.dacp_rayleigh_ritz(ctx, s["S"], s["P"], B_out=s["B"])
        # row j of the r x m block is column j of B
        return {"theta": theta, "B": _signed(s["B"].view(-1)[: r * case["m"]].view(r, case["m"]))}
    if op == "syev_batched":
        for w, a in zip(s["work"], s["A"]):  # the call destroys its matrices
            w.copy_(a)
        ws = B.dacp_syev_batched(ctx, s["work"], s["Z"])
        return {"w": ws, "Z": [_signed(z) for z in s["Z"]]}
    if op == "central":
        eigs, _, _, _ = B.dacp_central_eigs(ctx, s["ham"], case["N"], s["opts"])
        return eigs
    eigs, _, _, _, _ = B.dacp_central_eigs_batched(ctx, s["hams"], case["N"], s["opts"])
    return eigs


# ------------------------------------------------------------------ what a pass cannot do without

def _filter_order(case):
    return int(math.ceil(case["kfac"] / case["a_r"]))


def _steps(case):
    """Highest sampled order of the basis (the uniform grid's for the moment forms)."""
    if case["op"] == "basis":
        return 2 * int(math.floor(case["n"] * math.pi / (2.0 * case["a_r"])))
    return case["n"] * max(2, 2 * int(math.floor(math.pi / (2.0 * case["a_r"]))))


def _flips(model, L):
    """Off-diagonal Pauli strings of a model."""
    return {"chain": L, "glass": L, "tfim": L - 1, "sgs": L * (L - 1) // 2}[model]


def _call_work(model, L, N, b, o, moment):
    """A whole call's recurrences and dense solves, with the level density of a Gaussian spectrum."""
    D = float(1 << L)
    t = _terms(model, L, 1)
    sig = float(np.sqrt((t["coeff"] ** 2).sum()))
    e = _bound(model, L, 1)
    n_w = min(D, math.ceil(o.window_ratio * N))
    a_r = min(0.5, n_w * math.sqrt(2 * math.pi) * sig / (2 * D) / e)
    m = o.basis_ratio * n_w
    applies = b * (2 * o.kfac / a_r + (m / b - 1) / 2 * math.pi / a_r)
    flops = applies * 2 * D * (_flips(model, L) + 1)
    flops += 2 * D * m * (14 * b if moment else 2 * m) + 2 * D * m * N + 2 * (9.0 * m ** 3)
    return {"bytes": 8 * D * (m + N) + 32 * m * m, "flops": flops}


def work(case):
    op = case["op"]
    if op == "apply":
        D, b, w = 1 << case["L"], case["b"], 4 if case["dtype"] == "f32" else 8
        return {"bytes": w * D * (2 * b + 1), "flops": 2.0 * D * b * (_flips(case["model"], case["L"]) + 1)}
    if op == "estimates":
        D, f = 1 << case["L"], _flips(case["model"], case["L"]) + 1
        ap = case["steps"] + case["moments"] / 2 * case["nvec"]
        return {"bytes": 8.0 * D * (case["nvec"] + 2), "flops": 2.0 * D * ap * (f + 3)}
    if op == "filter":
        D, b = 1 << case["L"], case["b"]
        return {"bytes": 8.0 * D * (2 * b + 1),
                "flops": 2.0 * _filter_order(case) * 2 * D * b * (_flips(case["model"], case["L"]) + 2)}
    if op in ("basis", "stored", "moments"):
        D, b, k = 1 << case["L"], case["b"], _steps(case)
        m = b * (2 * case["n"] + 1)
        f = 2.0 * D * b * (_flips(case["model"], case["L"]) + 2)
        if op == "basis":
            return {"bytes": 8.0 * D * (b + m), "flops": k * f}
        if op == "stored":
            return {"bytes": 8.0 * (D * (b + m) + 2 * m * m), "flops": (k + 1) * f + 2.0 * D * 14 * b * m}
        # two b x b products at each of the grid's 3 (2 n + 1) or so recorded orders
        return {"bytes": 8.0 * (D * b + 2 * m * m), "flops": 2 * k * f + 6 * (2 * case["n"] + 1) * 2.0 * D * b * b}
    if op == "project":
        D, m = 1 << case["L"], case["m"]
        return {"bytes": 8.0 * (D * m + 2 * m * m), "flops": 2.0 * D * m * m}
    if op == "ritz":
        m = float(case["m"])
        r = case["rank"] * m
        # tridiagonal forms, back transformations, the reduction of P and the return to B
        return {"bytes": 8 * (2 * m * m + r * m), "flops": 4 / 3 * (m ** 3 + r ** 3) + 4 * (m * m * r + r ** 3) + 4 * r * m * m}
    if op == "syev_batched":
        ns = _batched_sizes(case)
        return {"bytes": 8.0 * sum(2 * n * n for n in ns), "flops": sum(16 / 3 * n ** 3 for n in ns)}
    if op == "central":
        o = _plain_opts(case)
        return _call_work(case["model"], case["L"], case["N"], case["b"], o, case["tuned"])
    o = _plain_opts(case)
    span = case["L_hi"] - case["L_lo"] + 1
    ws = [_call_work("glass", case["L_lo"] + i % span, case["N"], case["b"], o, case["tuned"]) for i in range(case["count"])]
    return {k: sum(w[k] for w in ws) for k in ("bytes", "flops")}


class _plain_opts:
    """The options that set a whole call's sizes (window_ratio, basis_ratio, kfac)."""

    def __init__(self, case):
        self.window_ratio, self.basis_ratio, self.kfac = 2.2, 1.5, 18.0
        if case["tuned"]:
            self.kfac = 12.0
            self.window_ratio, self.basis_ratio = (2.2, 1.3) if case["op"] == "batch" else (2.4, 1.2)


# ------------------------------------------------------------------ the same in plain 64-bit torch

class _Plain:
    """H as plain torch operations on [D][b] blocks."""

    def __init__(self, model, L, seed):
        s = torch.arange(1 << L, device=DEV)
        self.s, self.flips = s, {}
        self.d = torch.zeros(1 << L, device=DEV, dtype=torch.float64)
        for t in _terms(model, L, seed):
            x = z = ny = 0
            for op, site in ((int(t["op_a"]), int(t["site_a"])), (int(t["op_b"]), int(t["site_b"]))):
                if op in (inputs.X, inputs.Y):
                    x ^= 1 << site
                if op in (inputs.Z, inputs.Y):
                    z ^= 1 << site
                ny += op == inputs.Y
            c = float(t["coeff"]) * (-1.0 if ny == 2 else 1.0)
            if x == 0:
                self.d += c * self._sign(s, z)
            else:
                self.flips[(x, z)] = self.flips.get((x, z), 0.0) + c

    @staticmethod
    def _sign(s, z):
        p, v = torch.zeros_like(s), s & z
        while z:
            p ^= v & 1
            v, z = v >> 1, z >> 1
        return 1.0 - 2.0 * p.double()

    def __call__(self, v):
        y = self.d[:, None] * v
        for (x, z), c in self.flips.items():
            t = v[self.s ^ x]
            y.add_(t * self._sign(self.s ^ x, z)[:, None] if z else t, alpha=c)
        return y


def _exact_ritz(S, P, eps=1e-12):
    lam, U = np.linalg.eigh(S)
    keep = lam > eps
    U = U[:, keep] / np.sqrt(lam[keep])
    H = U.T @ P @ U
    theta, Y = np.linalg.eigh(0.5 * (H + H.T))
    return theta, (U @ Y).T


def _signed_np(z):
    big = np.take_along_axis(z, np.abs(z).argmax(axis=1)[:, None], 1)
    return z * np.where(big < 0, -1.0, 1.0)


def exact(case, seed):
    op = case["op"]
    if op == "ritz":
        S, P, _ = _pencil(case, seed)
        theta, b = _exact_ritz(S.cpu().numpy(), P.cpu().numpy())
        return {"theta": theta, "B": _signed_np(b)}
    if op == "syev_batched":
        g = _gen(seed)
        es = [np.linalg.eigh(_goe(n, g).cpu().numpy()) for n in _batched_sizes(case)]
        return {"w": [e[0] for e in es], "Z": [_signed_np(np.ascontiguousarray(e[1].T)) for e in es]}
    if op == "batch":
        return None
    model, L = case["model"], case["L"]
    D = 1 << L
    if op == "central":
        if L > 11:
            return None
        h = _Plain(model, L, seed)
        e = np.linalg.eigvalsh(h(torch.eye(D, device=DEV, dtype=torch.float64)).cpu().numpy())
        return np.sort(e[np.argsort(np.abs(e), kind="stable")[: case["N"]]])
    h = _Plain(model, L, seed)
    if op == "apply":
        x = _block(D, case["b"], seed, torch.float32 if case["dtype"] == "f32" else torch.float64)
        return h(x.double())
    if op == "estimates":
        return _exact_estimates(case, h, _block(D, 1, seed), _block(D, case["nvec"], seed + 1), _terms(model, L, seed))
    if op == "project":
        V = _block(D, case["m"], seed) / math.sqrt(D)
        P = torch.empty(case["m"], case["m"], device=DEV, dtype=torch.float64)
        for c in range(0, case["m"], 256):
            P[:, c:c + 256] = V.T @ h(V[:, c:c + 256].contiguous())
        return {"S": V.T @ V, "P": P}
    e = _bound(model, L, seed)
    a = case["a_r"] * e
    x = _unit_block(D, case["b"], seed)
    applies = 2 * _filter_order(case) if op == "filter" else _steps(case) * (2 if op == "moments" else 1)
    if applies * len(h.flips) * D * case["b"] > 1.5e12:  # over 20 seconds
        return None
    if op == "filter":
        ec, e0 = 0.5 * (e * e + a * a), 0.5 * (e * e - a * a)
        rho = math.exp(math.acosh(1.0 + 2.0 * a * a / (e * e - a * a)))
        t0, t1 = x, (h(h(x)) - ec * x) / (e0 * rho)
        for _ in range(1, _filter_order(case)):
            t0, t1 = t1, (h(h(t1)) - ec * t1) * (2.0 / (e0 * rho)) - t0 / (rho * rho)
        return t1 / t1.norm(dim=0)
    return _exact_basis(case, h, x, e, a)


def _exact_basis(case, h, x, e, a):
    b, n, op = case["b"], case["n"], case["op"]
    a_r = a / e
    if op == "basis":
        ks = [2 * int(math.floor(j * math.pi / (2.0 * a_r))) for j in range(1, n + 1)]
    else:
        d = max(2, 2 * int(math.floor(math.pi / (2.0 * a_r))))
        ks = [j * d for j in range(1, n + 1)]
    at = {0: 0}
    for j, k in enumerate(ks):
        at[k - 1], at[k] = 2 * j + 1, 2 * j + 2
    V = torch.zeros(x.shape[0], b * (2 * n + 1), device=DEV, dtype=torch.float64)
    t0, t1 = x, h(x) / e
    V[:, :b] = x
    for k in range(1, ks[-1] + 1):
        if k in at:
            V[:, at[k] * b:(at[k] + 1) * b] = t1
        t0, t1 = t1, h(t1) * (2.0 / e) - t0
    if op == "basis":
        return V
    S, P = V.T @ V, V.T @ h(V)
    return {"V": V, "S": S, "P": P} if op == "stored" else {"S": S, "P": P}


def _exact_estimates(case, h, v, R, terms):
    v, vp, beta, al, be = v / v.norm(), torch.zeros_like(v), 0.0, [], []
    for _ in range(case["steps"]):
        w = h(v) - beta * vp
        al.append(float((w * v).sum()))
        w = w - al[-1] * v
        beta = float(w.norm())
        be.append(beta)
        v, vp = w / beta, v
    t, y = np.linalg.eigh(np.diag(al) + np.diag(be[:-1], 1) + np.diag(be[:-1], -1))
    r = np.abs(be[-1] * y[-1])
    e = min(1.01 * max(abs(t[-1]) + r[-1], abs(t[0]) + r[0]), float(np.abs(terms["coeff"]).sum()))
    mu = np.zeros(case["moments"])
    n0 = float((R * R).sum())
    t0, t1 = R, h(R) / e
    mu[0], mu[1] = 1.0, float((R * t1).sum()) / n0
    for k in range(2, case["moments"]):
        t0, t1 = t1, h(t1) * (2.0 / e) - t0
        mu[k] = float((R * t1).sum()) / n0
    return {"bound": np.array([e, t[0], t[-1]]), "mu": mu}
