"""The pivoting panel run by a team of workgroups (one row a thread, rows of a shift spread
over workgroups) against the panel run by one workgroup from memory, and against the
spectrum, where its sizes are at an edge: one workgroup's rows and one more, the narrow and
the wide panel, the last panel, one column."""
import numpy as np
import pytest
import torch

from paper_1908_06043_amd import inputs
from tests.gpu_helpers import backward_error, decode_factor, inertia_of

pytestmark = pytest.mark.gpu
U = np.finfo(np.float64).eps / 2


def dev(M):
    return torch.from_numpy(np.ascontiguousarray(M)).cuda()


def _matrix(kind, n):
    C = inputs.random_symmetric(n, n + 40)
    if kind == "two_by_two":          # zero diagonal: 2x2 pivots and interchanges
        np.fill_diagonal(C, 0.0)
    elif kind == "ties":              # small integers: equal maxima, the lowest row wins
        C = np.round(1.5 * C)
        C = 0.5 * (C + C.T) + np.diag(np.full(n, 1.0 / 3.0))
    return C


@pytest.mark.parametrize("kind", ["random", "two_by_two", "ties"])
@pytest.mark.parametrize("n", [2, 33, 63, 1023, 1024, 1025, 2048, 2049, 2570])
def test_team_panel_backward_error_and_inertia(gpu_lib, kind, n):
    C = _matrix(kind, n)
    f = gpu_lib.ldlt_factor(dev(C), dev(np.eye(n)), 0.0)
    w = np.linalg.eigvalsh(C)
    assert f.inertia == (int(np.sum(w < 0)), 0, int(np.sum(w > 0)))
    LD, ip = f.LD.cpu().numpy(), f.ipiv.cpu().numpy()
    assert backward_error(C, LD, ip) <= 100 * n * U   # the bound of the other factor tests
    L, D, perm, blocks = decode_factor(LD, ip)
    assert inertia_of(D) == f.inertia


@pytest.mark.parametrize("kind", ["random", "two_by_two", "ties"])
def test_team_equals_one_workgroup_bitwise(gpu_lib, kind):
    """48 shifts of order 2100 need more workgroups than run at once, so their panels run
    from memory, one workgroup a shift, until enough rows are done; one shift alone runs as
    a team of five from the start.  The operations and their order are the same."""
    n = 2100
    A, I = dev(_matrix(kind, n)), dev(np.eye(n))
    sig = [float(s) for s in np.linspace(-31.0, 29.0, 48)]
    facs = gpu_lib.ldlt_factor_multi(A, I, sig)
    for k in (0, 17, 24, 47):
        g = gpu_lib.ldlt_factor(A, I, sig[k])
        assert g.inertia == facs[k].inertia
        assert torch.equal(g.ipiv, facs[k].ipiv)
        assert torch.equal(torch.tril(g.LD), torch.tril(facs[k].LD))


@pytest.mark.parametrize("kind", ["random", "two_by_two"])
@pytest.mark.parametrize("n", [255, 256, 257, 511, 512, 513, 1090, 1537])
def test_one_workgroup_panels_of_every_size(gpu_lib, kind, n):
    """Panels of at most 256, 512 and 1024 rows run on as many threads; an order between them
    passes every smaller size on its way down, narrow panels (those of every order here) on one workgroup or two."""
    C = _matrix(kind, n)
    f = gpu_lib.ldlt_factor(dev(C), dev(np.eye(n)), 0.0)
    w = np.linalg.eigvalsh(C)
    assert f.inertia == (int(np.sum(w < 0)), 0, int(np.sum(w > 0)))
    assert backward_error(C, f.LD.cpu().numpy(), f.ipiv.cpu().numpy()) <= 100 * n * U
