"""One factor applied to blocks of right-hand sides: the sweeps run groups of 16 columns
side by side, and the preparation forms the look-ahead blocks with or without a
workgroup of its own for each (few or many row blocks).  Checked at the edges of the
groups and of the 64-row blocks, with 2x2 pivots that straddle a block border and runs of
them longer than a block."""
import numpy as np
import pytest
import torch

from paper_1908_06043_amd import inputs

pytestmark = pytest.mark.gpu


def dev(M):
    return torch.from_numpy(np.ascontiguousarray(M)).cuda()


def _pairs(n, seed):
    """Coupled pairs [[0, 1], [1, 0]] behind one ordinary row, weakly perturbed with a
    zero diagonal: Bunch-Kaufman takes 2x2 pivots throughout, at odd offsets."""
    C = 0.02 / np.sqrt(n) * inputs.random_symmetric(n, seed)
    np.fill_diagonal(C, 0.0)
    C[0, 0] = 2.0
    for i in range(1, n - 1, 2):
        C[i, i + 1] = C[i + 1, i] = 1.0 + 0.001 * i / n
    if n % 2 == 0:
        C[-1, -1] = 3.0
    return C


@pytest.mark.parametrize("kind", ["random", "pairs"])
@pytest.mark.parametrize("n", [1, 63, 64, 129, 200, 321])
@pytest.mark.parametrize("nrhs", [1, 16, 17, 33, 64])
def test_groups_of_right_hand_sides(gpu_lib, kind, n, nrhs):
    C = inputs.random_symmetric(n, n) if kind == "random" else _pairs(n, n)
    f = gpu_lib.ldlt_factor(dev(C), dev(np.eye(n)), 0.0)
    if kind == "pairs" and n > 64:
        neg = f.ipiv.cpu().numpy() < 0
        assert neg[1:64].all() or neg.mean() > 0.9   # long runs of 2x2 rows
    Y = np.random.default_rng(n + nrhs).standard_normal((n, nrhs))
    X = gpu_lib.ldlt_solve(f, dev(Y)).cpu().numpy()
    r = np.linalg.norm(C @ X - Y) / (np.linalg.norm(C) * np.linalg.norm(X))
    assert r < 1e-13   # the bound of the other solve tests
    # a column does not depend on the group it runs in
    one = gpu_lib.ldlt_solve(f, dev(Y[:, nrhs - 1])).cpu().numpy()
    assert np.array_equal(one, X[:, nrhs - 1])


def test_many_row_blocks(gpu_lib):
    """More than 128 row blocks: one workgroup forms all four look-ahead products, and
    the row blocks of the one factor are shared out over every XCD."""
    n = 8257
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    G = torch.randn((n, n), generator=g, dtype=torch.float64, device="cuda")
    C = (0.5 * (G + G.T)).contiguous()
    f = gpu_lib.ldlt_factor(C, torch.eye(n, dtype=torch.float64, device="cuda"), 0.0)
    Y = torch.randn((n, 20), generator=g, dtype=torch.float64, device="cuda")
    X = gpu_lib.ldlt_solve(f, Y)
    r = torch.linalg.norm(C @ X - Y) / (torch.linalg.norm(C) * torch.linalg.norm(X))
    assert float(r) < 1e-13
