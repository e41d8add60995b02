"""A shift that all but coincides with an eigenvalue: the vectors of the probe's first steps
are then 1 / distance long, and their rounding must not end up in the other eigenvectors'
residuals.  Planned shifts come this close now and then (1e-6 once in 500 pencils), so the
bar is the plain path's: status OK, eigenvalues within 1e-10 max|lambda| of the
construction's spectrum, residuals at most 1e-10, B-orthonormal vectors."""
import numpy as np
import pytest
import torch

from paper_1908_06043_amd import inputs

pytestmark = pytest.mark.gpu


def _pencil(n, seed):
    lam = lambda r, k: inputs.spectrum_scf(r, k, n // 10)
    return inputs.make_pencil_device(n, lam, seed, "cuda")


def _check(out, A, B, lam, n_e):
    assert out["status"] == 0, (out["status"], float(out["resid"].max()))
    assert np.max(np.abs(out["evals"].cpu().numpy() - lam[:n_e])) <= 1e-10 * np.max(np.abs(lam))
    assert float(out["resid"].max()) <= 1e-10
    X = out["evecs"]
    G = (X.T @ (B @ X)).cpu().numpy()
    assert np.max(np.abs(G - np.eye(n_e))) <= 1e-10


@pytest.mark.parametrize("n,seed", [(512, 1), (950, 2), (1536, 3)])
@pytest.mark.parametrize("probe", [0, 2, 5, 7])
@pytest.mark.parametrize("d", [3e-5, 1e-6, -1e-7, 1e-8, -1e-9,
                               # the Gram matrix of the first block has condition 1e20 and its
                               # Cholesky factorization breaks down: missing eigenvalues reported
                               pytest.param(1e-10, marks=pytest.mark.xfail(strict=False, reason="block collapses"))])
def test_shift_next_to_an_eigenvalue(gpu_lib, n, seed, probe, d):
    n_e = n // 10
    A, B, lam = _pencil(n, seed)
    plan = gpu_lib.plan_shifts_kpm(A, B, n_e, 8)
    sig, top = plan["sigmas"].copy(), plan["omega_top"]
    k = int(np.argmin(np.abs(lam - sig[probe])))
    sig[probe] = lam[k] + d
    assert np.all(np.diff(sig) > 0) and sig[-1] < top
    print(f"n={n} probe={probe} d={d}", flush=True)
    out = gpu_lib.solve(A, B, n_e, 8, sigmas=sig, omega_top=top, check=False)
    _check(out, A, B, lam, n_e)


def test_several_shifts_next_to_eigenvalues(gpu_lib):
    """Every shift at once, and pairs of eigenvalues next to one shift."""
    n, n_e = 700, 70
    A, B, lam = inputs.make_pencil_device(n, lambda r, k: _paired(r, k), 11, "cuda")
    sig = np.array([lam[2 * j + 8 * j] + 3e-8 for j in range(7)])
    out = gpu_lib.solve(A, B, n_e, 7, sigmas=sig, omega_top=0.5 * (lam[n_e + 3] + lam[n_e + 4]), check=False)
    _check(out, A, B, lam, n_e)


def _paired(rng, n):
    """Eigenvalues in pairs 1e-6 apart."""
    v = np.sort(rng.uniform(-5.0, 5.0, n // 2))
    return np.sort(np.concatenate([v, v + 1e-6]))
