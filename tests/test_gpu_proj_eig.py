"""The eigensolver of the solve path's projected problems (reduction to tridiagonal form and
divide and conquer) against LAPACK, at the orders where its segments, 8-lane groups and
16-wide tiles are ragged, and on spectra that deflate: repeated and nearly equal
eigenvalues, decoupled blocks, the thick-restart shape, extreme scales."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

ORDERS = [1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 23, 31, 32, 33, 48, 49, 56, 57, 63, 64, 65, 80, 96, 97, 100, 111, 112]


def _matrix(kind, m, rng):
    G = rng.standard_normal((m, m))
    S = 0.5 * (G + G.T)
    if kind == "random":
        return S
    if kind == "diagonal":
        return np.diag(np.round(rng.uniform(-3, 3, m), 1))
    if kind == "zero":
        return np.zeros((m, m))
    if kind == "near_identity":      # the B-Gram matrix of locked vectors
        return np.eye(m) + 1e-14 * S
    if kind == "repeated":
        Q, _ = np.linalg.qr(G)
        lam = np.repeat(rng.uniform(-5, 5, m // 4 + 1), 4)[:m]
        M = (Q * lam) @ Q.T
        return 0.5 * (M + M.T)
    if kind == "clustered":          # pairs 1e-13 apart
        Q, _ = np.linalg.qr(G)
        lam = np.repeat(rng.uniform(-5, 5, m // 2 + 1), 2)[:m] + 1e-13 * np.arange(m)
        M = (Q * lam) @ Q.T
        return 0.5 * (M + M.T)
    if kind == "restart":            # kept Ritz values, their coupling, banded new blocks
        k = max(1, (7 * m) // 10)
        T = np.diag(np.concatenate([1.0 / rng.uniform(-0.3, 0.3, k), rng.uniform(-10, 10, m - k)]))
        hi = min(m, k + 8)
        C = rng.standard_normal((hi - k, k)) * 10.0 ** rng.uniform(-12, 0, k)
        T[k:hi, :k] = C
        T[:k, k:hi] = C.T
        for i in range(k, m):
            for j in range(k, i):
                if i - j <= 8:
                    T[i, j] = T[j, i] = rng.standard_normal()
        return T
    if kind == "wilkinson":          # eigenvalues in pairs that agree to working precision
        T = np.diag(np.abs(np.arange(m) - (m - 1) / 2.0))
        return T + np.diag(np.ones(m - 1), 1) + np.diag(np.ones(m - 1), -1)
    return S * {"tiny": 1e-200, "huge": 1e200}[kind]


@pytest.mark.parametrize("kind", ["random", "diagonal", "zero", "near_identity", "repeated", "clustered",
                                  "restart", "wilkinson", "tiny", "huge"])
def test_proj_eig_matches_lapack(gpu_lib, kind):
    rng = np.random.default_rng(len(kind))
    mats = [_matrix(kind, m, rng) for m in ORDERS]
    out = gpu_lib.proj_eig([torch.from_numpy(x).cuda() for x in mats])
    for x, (W, V) in zip(mats, out):
        m = x.shape[0]
        W, V = W.cpu().numpy(), V.cpu().numpy()
        ref = np.linalg.eigvalsh(x)
        scale = max(np.abs(ref).max(), 1e-300)
        # the bounds of the Jacobi solver's tests
        assert np.all(np.diff(W) >= 0), (kind, m)
        assert np.max(np.abs(W - ref)) <= 1e-13 * scale, (kind, m)
        assert np.max(np.abs(V.T @ V - np.eye(m))) <= 1e-13, (kind, m)
        assert np.max(np.abs((x / scale) @ V - V * (W / scale)[None, :])) <= 1e-13, (kind, m)
