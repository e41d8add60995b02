"""The library's work as its users call it, for timing and for comparing results.

A case names one public call (``op``) and its sizes:

* ``factor``: ``api.ldlt_factor_multi``, the Bunch-Kaufman factors and inertias of
  A - sigma B for a set of shifts;
* ``apply``: ``api.ldlt_solve``, right-hand sides through factors the program holds;
* ``plan``: ``api.plan_shifts_kpm``, the density-of-states shift placement;
* ``solve``: ``api.solve``, planning and the lowest n_e eigenpairs of one pencil; an SCF
  program goes on with the eigenvalues and the density matrix of the eigenvectors;
* ``grad``: ``api.eigh_pencil`` forward and backward on a density-matrix loss;
* ``batch``: ``api.solve_batched`` on pencils of uneven order.

The pencils are the SCF-shaped ones of the benchmark (12 clusters on a uniform
background in [-5, 5], two gaps, B close to the identity with exponentially decaying
overlaps), built from their eigenpairs so that every result is known.
"""
import math

import numpy as np
import torch

from paper_1908_06043_amd import api

F64 = dict(dtype=torch.float64, device="cuda")
GAP = 0.05   # between the wanted eigenvalues and the rest: the density matrix is defined


def listed():
    return [
        # one shift of the smallest pencil in use (N = 200): latency and launches
        dict(name="factor_n200", op="factor", n=200, shifts=1),
        # a mid-sized pencil of odd order, a handful of shifts
        dict(name="factor_n1001_s5", op="factor", n=1001, shifts=5),
        # the factorization phase of the plain workload: 16 shifts and the top boundary
        dict(name="factor_n4096_s17", op="factor", n=4096, shifts=17),
        # the SCF order, one rank's share of the shifts
        dict(name="factor_n12288_s8", op="factor", n=12288, shifts=8),
        # one vector through small factors, as an outer iteration calls it
        dict(name="apply_n200_r1", op="apply", n=200, nrhs=1),
        # a full-width block of right-hand sides, ragged order
        dict(name="apply_n2501_r64", op="apply", n=2501, nrhs=64),
        # one Lanczos block through large factors
        dict(name="apply_n8192_r8", op="apply", n=8192, nrhs=8),
        # shift placement alone, as a program plans once for several solves
        dict(name="plan_n2048", op="plan", n=2048, n_e=200, n_s=8),
        # a small whole solve
        dict(name="solve_n1000", op="solve", n=1000, n_e=100, n_s=4),
        # the plain workload: N = 4096, n_e = 400, 16 shifts
        dict(name="solve_n4096", op="solve", n=4096, n_e=400, n_s=16),
        # the differentiated workload: N = 2048, n_e = 200, 8 shifts, both gradients
        dict(name="grad_n2048", op="grad", n=2048, n_e=200, n_s=8),
        # many small pencils at once, orders spread as in the batched workload's lower half
        dict(name="batch_8", op="batch", count=8, lo=512, hi=1536, n_s=8),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["factor", "factor", "factor", "apply", "apply", "apply", "plan", "solve", "solve", "grad", "batch"])
    if op == "factor":
        n = _log(rng, 64, 12288)
        most = min(17, 8 * (12288 / n) ** 3)   # no more work than the largest listed one
        return dict(op=op, n=n, shifts=min(17, max(1, _log(rng, 1, most))))
    if op == "apply":
        return dict(op=op, n=_log(rng, 64, 8192), nrhs=_log(rng, 1, 64))
    if op == "batch":
        lo = 64 * rng.randint(5, 9)
        return dict(op=op, count=rng.randint(4, 8), lo=lo, hi=lo + 32 * rng.randint(8, 30), n_s=8)
    n = _log(rng, 300, 2048 if op == "grad" else 4096)
    n_e = max(24, int(n * rng.uniform(0.06, 0.1)))
    return dict(op=op, n=n, n_e=n_e, n_s=min(16, max(2, round(n_e / rng.uniform(16, 26)))))


# ------------------------------------------------------------------ pencils

def _spectrum(n, n_e, seed):
    """Half uniform on [-5, 5], half in 12 clusters of width 0.05; two windows of width
    0.1 empty inside the wanted part; GAP above the n_e-th value."""
    r = np.random.default_rng([int(seed), n, 1])
    centres = r.uniform(-5.0, 5.0, 12)

    def some(m):
        c = centres[r.integers(0, 12, m)]
        return np.where(r.random(m) < 0.5, r.uniform(-5.0, 5.0, m), r.normal(c, 0.05))

    v = np.clip(some(n), -5.0, 5.0)
    s = np.sort(v)
    holes = s[0] + (s[n_e - 1] - s[0]) * np.array([1.0, 2.0]) / 3.0
    for _ in range(200):
        bad = (np.abs(v) >= 5.0) | (np.abs(v[:, None] - holes[None, :]) < 0.05).any(1)
        if not bad.any():
            break
        v[bad] = some(int(bad.sum()))
    lam = np.sort(v)
    lam[n_e:] += max(0.0, GAP - (lam[n_e] - lam[n_e - 1]))
    return lam


def _pencil(n, n_e, seed):
    """A = L Q diag(lam) Q^T L^T and B = L L^T: eigenvalues lam, eigenvectors L^-T Q.
    L is unit lower triangular with decaying entries, Q two sign flips between three
    Hartley transforms (orthogonal, entries as of a random rotation)."""
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 131 + n)

    def hartley(x):
        f = torch.fft.fft(x, dim=0)
        return (f.real - f.imag) / math.sqrt(n)

    lam = _spectrum(n, n_e, seed)
    i = torch.arange(n, **F64)
    L = torch.randn((n, n), generator=g, **F64)
    L *= 0.05 * torch.exp(-(i[:, None] - i[None, :]).abs() / 5.0)
    L = torch.tril(L, -1)
    L.diagonal().fill_(1.0)
    Q = hartley(torch.eye(n, **F64))
    for _ in range(2):
        flip = torch.randint(0, 2, (n, 1), generator=g, **F64) * 2.0 - 1.0
        Q = hartley(flip * Q)
    A = L @ ((Q * torch.from_numpy(lam).cuda()[None, :]) @ Q.T) @ L.T
    A = (0.5 * (A + A.T)).contiguous()
    B = L @ L.T
    B = (0.5 * (B + B.T)).contiguous()
    return dict(A=A, B=B, lam=lam, L=L, Q=Q, g=g)


def _shifts(lam, n_e, count):
    """Shifts spread over the wanted values, each in the widest gap near its place."""
    out = []
    for j in range(count):
        lo, hi = j * n_e // count, max((j + 1) * n_e // count, j * n_e // count + 1)
        k = lo + int(np.argmax(lam[lo + 1:hi + 1] - lam[lo:hi]))
        out.append(0.5 * (lam[k] + lam[k + 1]))
    return np.array(out)


def _wanted(case):
    return max(8, case["n"] // 10) if case["op"] in ("factor", "apply") else case["n_e"]


def _weight(n, g):
    G = torch.randn((n, n), generator=g, **F64)
    return ((G + G.T) / math.sqrt(2.0)).contiguous()


def _orders(case):
    """Orders of a batch, from lo to hi."""
    c = case["count"]
    return [case["lo"] + (case["hi"] - case["lo"]) * i // (c - 1) for i in range(c)]


# ------------------------------------------------------------------ the cases

def prepare(case, seed):
    op = case["op"]
    if op == "batch":
        ps = [_pencil(n, n // 10, seed * 64 + i) for i, n in enumerate(_orders(case))]
        return dict(op=op, pencils=[(p["A"], p["B"], p["A"].shape[0] // 10, case["n_s"]) for p in ps])
    n_e = _wanted(case)
    p = _pencil(case["n"], n_e, seed)
    s = dict(op=op, A=p["A"], B=p["B"], n_e=n_e)
    if op == "factor":
        s["sigmas"] = _shifts(p["lam"], n_e, case["shifts"])
    elif op == "apply":
        # a program that applies C^-1 holds the factors of its shift
        s["factor"] = api.ldlt_factor(p["A"], p["B"], float(_shifts(p["lam"], n_e, 2)[1]))
        s["rhs"] = torch.randn((case["n"], case["nrhs"]), generator=p["g"], **F64)
        del s["A"], s["B"]
    else:
        s["n_s"] = case["n_s"]
        if op == "grad":
            s["W"] = _weight(case["n"], p["g"])
    return s


def run(s):
    op = s["op"]
    if op == "factor":
        fs = api.ldlt_factor_multi(s["A"], s["B"], s["sigmas"])
        # L and D are the lower triangle (LDt is stored transposed)
        return dict(LD=[f.LDt.triu_() for f in fs], ipiv=[f.ipiv for f in fs],
                    inertia=np.array([f.inertia for f in fs]))
    if op == "apply":
        return api.ldlt_solve(s["factor"], s["rhs"])
    if op == "plan":
        return api.plan_shifts_kpm(s["A"], s["B"], s["n_e"], s["n_s"])
    if op == "solve":
        out = api.solve(s["A"], s["B"], s["n_e"], s["n_s"])
        X = out["evecs"]
        return dict(evals=out["evals"], density=X @ X.T, nu=out["report"]["nu"])
    if op == "grad":
        A, B = s["A"].detach().requires_grad_(True), s["B"].detach().requires_grad_(True)
        lam, X = api.eigh_pencil(A, B, s["n_e"], s["n_s"])
        loss = lam.square().sum() + (s["W"] * (X @ X.T)).sum()
        GA, GB = torch.autograd.grad(loss, (A, B))
        return dict(evals=lam.detach(), loss=loss.detach(), GA=GA, GB=GB)
    outs, _ = api.solve_batched(s["pencils"])
    return [dict(evals=o["evals"], density=o["evecs"] @ o["evecs"].T) for o in outs]


def work(case):
    op = case["op"]
    if op == "batch":
        each = [work(dict(op="solve", n=n, n_e=n // 10, n_s=case["n_s"])) for n in _orders(case)]
        return {k: sum(e[k] for e in each) for k in ("bytes", "flops")}
    n = float(case["n"])
    tri = 4.0 * n * n                       # bytes of one triangle in FP64
    if op == "factor":
        S = case["shifts"]
        return dict(bytes=2 * tri + S * (tri + 4 * n), flops=S * n ** 3 / 3)
    if op == "apply":
        return dict(bytes=tri + 16 * n * case["nrhs"], flops=2 * n * n * case["nrhs"])
    # 32 applications of the operator (A and two triangular solves) to 20 vectors give
    # 64 moments, after one factorization of B
    plan = n ** 3 / 3 + 32 * 20 * 4 * n * n
    if op == "plan":
        return dict(bytes=2 * tri, flops=plan)
    n_e, n_s = case["n_e"], case["n_s"]
    # one factorization a shift and boundary; each wanted vector through one solve and
    # one product with A and with B
    solve = plan + (n_s + 1) * n ** 3 / 3 + 6 * n * n * n_e + 2 * n * n * n_e
    if op == "solve":
        return dict(bytes=2 * tri + 8 * n * n_e + 8 * n * n, flops=solve)
    # backward: the cotangent, one solve a vector and two symmetric rank-2n_e products
    return dict(bytes=2 * tri + 24 * n * n, flops=solve + 6 * n * n * n_e + 4 * n * n * n_e)


def _density(p, n_e):
    X = torch.linalg.solve_triangular(p["L"].T, p["Q"][:, :n_e].contiguous(), upper=True, unitriangular=True)
    return X @ X.T


def exact(case, seed):
    op = case["op"]
    if op == "batch":
        out = []
        for i, n in enumerate(_orders(case)):
            p = _pencil(n, n // 10, seed * 64 + i)
            out.append(dict(evals=p["lam"][:n // 10], density=_density(p, n // 10)))
        return out
    n, n_e = case["n"], _wanted(case)
    p = _pencil(n, n_e, seed)
    lam = p["lam"]
    if op == "factor":
        # the counts below each shift; the factors themselves depend on the pivots taken
        sig = _shifts(lam, n_e, case["shifts"])
        neg = [int(np.sum(lam < x)) for x in sig]
        S = case["shifts"]
        return dict(LD=[None] * S, ipiv=[None] * S, inertia=np.array([(k, 0, n - k) for k in neg]))
    if op == "apply":
        C = p["A"] - float(_shifts(lam, n_e, 2)[1]) * p["B"]
        rhs = torch.randn((n, case["nrhs"]), generator=p["g"], **F64)
        x = torch.linalg.solve(C, rhs)
        return x + torch.linalg.solve(C, rhs - C @ x)
    if op == "plan":
        return None   # a stochastic estimate from the library's own random vectors
    if op == "solve":
        return dict(evals=lam[:n_e], density=_density(p, n_e), nu=None)
    W = _weight(n, p["g"])
    X = torch.linalg.solve_triangular(p["L"].T, p["Q"], upper=True, unitriangular=True)
    l = torch.from_numpy(lam).cuda()
    T = X.T @ W @ X
    KA, KB = torch.zeros_like(T), torch.zeros_like(T)
    # wanted against the rest: dD carries T_ia (dA_ia - lam_i dB_ia) / (lam_i - lam_a)
    K = T[:n_e, n_e:] / (l[:n_e, None] - l[None, n_e:])
    KA[:n_e, n_e:], KA[n_e:, :n_e] = K, K.T
    K = -l[:n_e, None] * K
    KB[:n_e, n_e:], KB[n_e:, :n_e] = K, K.T
    # inside the wanted space only the normalisation and the eigenvalues move
    KB[:n_e, :n_e] = -T[:n_e, :n_e]
    KA.diagonal()[:n_e] += 2 * l[:n_e]
    KB.diagonal()[:n_e] -= 2 * l[:n_e] ** 2
    loss = l[:n_e].square().sum() + T.diagonal()[:n_e].sum()
    return dict(evals=l[:n_e].clone(), loss=loss, GA=X @ KA @ X.T, GB=X @ KB @ X.T)
