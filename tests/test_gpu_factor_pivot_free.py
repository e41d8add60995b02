"""The pivot-free panel where its sizes are at an edge (the diagonal block's last columns, one
wavefront's and one workgroup's rows below it, more rows than workgroups), and where one entry
far below the block decides: that column is rejected and the pivoting panel takes over."""
import numpy as np
import pytest
import torch

from paper_1908_06043_amd import inputs
from tests.gpu_helpers import backward_error, decode_factor, inertia_of

pytestmark = pytest.mark.gpu
U = np.finfo(np.float64).eps / 2


def dev(M):
    return torch.from_numpy(np.ascontiguousarray(M)).cuda()


def _dominant(n):
    C = inputs.random_symmetric(n, n + 7)
    sign = np.where(np.arange(n) % 3 == 0, -1.0, 1.0)
    return C + np.diag(sign * 4.0 * (1.0 + np.abs(C).sum(axis=1)))


def _check(lib, C):
    n = C.shape[0]
    f = lib.ldlt_factor(dev(C), dev(np.eye(n)), 0.0)
    w = np.linalg.eigvalsh(C)
    assert f.inertia == (int(np.sum(w < 0)), 0, int(np.sum(w > 0)))
    LD, ip = f.LD.cpu().numpy(), f.ipiv.cpu().numpy()
    assert backward_error(C, LD, ip) <= 100 * n * U   # the bound of the other factor tests
    L, D, perm, blocks = decode_factor(LD, ip)
    assert inertia_of(D) == f.inertia
    return ip


@pytest.mark.parametrize("n", [1, 7, 8, 9, 31, 32, 33, 40, 95, 96, 97, 287, 288, 289, 2049, 2113, 2369])
def test_dominant_matrix_takes_no_interchange(gpu_lib, n):
    ip = _check(gpu_lib, _dominant(n))
    assert np.array_equal(ip, np.arange(n)) or np.array_equal(ip, np.arange(1, n + 1))


@pytest.mark.parametrize("n,row,col", [(300, 33, 31), (300, 95, 0), (300, 96, 17), (300, 299, 30),
                                       (700, 288, 5), (700, 699, 31), (2200, 2199, 63), (2200, 319, 8)])
def test_one_large_entry_below_the_block(gpu_lib, n, row, col):
    C = _dominant(n)
    C[row, col] = C[col, row] = 1e3 * np.abs(C).max()
    ip = _check(gpu_lib, C)
    assert not (np.array_equal(ip, np.arange(n)) or np.array_equal(ip, np.arange(1, n + 1)))


@pytest.mark.parametrize("shifts", [300])
def test_more_shifts_than_workgroups_a_shift(gpu_lib, shifts):
    """With this many shifts each has one workgroup for all its rows."""
    n = 420
    C = _dominant(n)
    sig = [float(s) for s in np.linspace(-1.0, 1.0, shifts)]
    facs = gpu_lib.ldlt_factor_multi(dev(C), dev(np.eye(n)), sig)
    for k in (0, 151, shifts - 1):
        g = gpu_lib.ldlt_factor(dev(C), dev(np.eye(n)), sig[k])
        assert torch.equal(g.ipiv, facs[k].ipiv)
        assert torch.equal(torch.tril(g.LD), torch.tril(facs[k].LD))


@pytest.mark.parametrize("rows", [[], [0], [1], [2, 3], [5, 8, 9], [6], [7, 19], [0, 1, 2, 3, 4, 5, 6, 7, 8], [31]])
def test_waiting_updates_equal_single_ones_bitwise(gpu_lib, rows):
    """17 shifts of order 2600 are large enough (down to 1987 rows) for whole panels to wait for one another, one
    shift alone is not.  The panels named get an entry that needs pivoting, so that rows of
    waiting panels are completed, caught up, left at the end or never begun."""
    n, S = 2600, 17
    C = _dominant(n)
    for p in rows:
        i, j = 64 * p + 11, min(64 * p + 900, n - 1)
        C[i, j] = C[j, i] = 1e3 * np.abs(C).max()
    A, I = dev(C), dev(np.eye(n))
    sig = [float(s) for s in np.linspace(-3.0, 3.0, S)]
    facs = gpu_lib.ldlt_factor_multi(A, I, sig)
    for k in (0, 9, S - 1):
        g = gpu_lib.ldlt_factor(A, I, sig[k])
        assert g.inertia == facs[k].inertia
        assert torch.equal(g.ipiv, facs[k].ipiv)
        assert torch.equal(torch.tril(g.LD), torch.tril(facs[k].LD))
    f = facs[9]
    B = C - sig[9] * np.eye(n)
    assert backward_error(B, f.LD.cpu().numpy(), f.ipiv.cpu().numpy()) <= 100 * n * U


@pytest.mark.parametrize("n,zero", [(200, 0), (200, 31), (200, 32), (300, 299), (2100, 64), (2100, 100)])
def test_singular_b_is_refused(gpu_lib, n, zero):
    """B's factorization takes no interchange: a zero pivot ends the accepted columns and the
    panel goes on column by column; the planner refuses the pencil."""
    A = inputs.random_symmetric(n, n + 1)
    B = np.eye(n)
    B[zero, zero] = 0.0
    with pytest.raises(Exception, match="invalid argument"):
        gpu_lib.plan_shifts_kpm(dev(A), dev(B), n // 10, 4)
