"""The bound of the device-side waits and the factorization.  Below 2^16 polls no team of
workgroups gathers: the first workgroup of a pivoting panel runs it alone, which is also what
it does when the device is busy, so these tests compare that route with the team, bit for
bit (the operations and their order are the same).  A factorization captured under one bound
does not keep it."""
import numpy as np
import pytest
import torch

from paper_1908_06043_amd import inputs
from paper_1908_06043_amd._lib import SisliceError

pytestmark = pytest.mark.gpu
DEFAULT = 1 << 21


def dev(M):
    return torch.from_numpy(np.ascontiguousarray(M)).cuda()


def _limited(lib, polls, call):
    lib.set_wait_limit(polls)
    try:
        return call()
    finally:
        lib.set_wait_limit(DEFAULT)


def _same(f, g):
    assert f.inertia == g.inertia
    assert torch.equal(f.ipiv, g.ipiv)
    assert torch.equal(torch.tril(f.LD), torch.tril(g.LD))


def _matrix(kind, n):
    C = inputs.random_symmetric(n, n + 40)
    if kind == "two_by_two":          # zero diagonal: 2x2 pivots and interchanges
        np.fill_diagonal(C, 0.0)
    elif kind == "ties":              # small integers: equal maxima, the lowest row wins
        C = np.round(1.5 * C)
        C = 0.5 * (C + C.T) + np.diag(np.full(n, 1.0 / 3.0))
    return C


@pytest.mark.parametrize("kind", ["random", "two_by_two", "ties"])
@pytest.mark.parametrize("n", [1025, 1600, 2049, 2570])   # teams of two to six, 32 and 64 columns
@pytest.mark.parametrize("polls", [0, 3])
def test_first_workgroup_alone_equals_the_team(gpu_lib, kind, n, polls):
    A, I = dev(_matrix(kind, n)), dev(np.eye(n))
    _same(_limited(gpu_lib, polls, lambda: gpu_lib.ldlt_factor(A, I, 0.0)), gpu_lib.ldlt_factor(A, I, 0.0))


def test_first_workgroup_alone_with_waiting_updates(gpu_lib):
    """17 shifts of order 2600: whole panels wait for one another until one needs pivoting."""
    n = 2600
    C = inputs.random_symmetric(n, n + 7)
    sign = np.where(np.arange(n) % 3 == 0, -1.0, 1.0)
    C += np.diag(sign * 4.0 * (1.0 + np.abs(C).sum(axis=1)))
    for p in (2, 3, 7):
        i, j = 64 * p + 11, 64 * p + 900
        C[i, j] = C[j, i] = 1e3 * np.abs(C).max()
    A, I = dev(C), dev(np.eye(n))
    sig = [float(s) for s in np.linspace(-3.0, 3.0, 17)]
    alone = _limited(gpu_lib, 0, lambda: gpu_lib.ldlt_factor_multi(A, I, sig))
    for f, g in zip(alone, gpu_lib.ldlt_factor_multi(A, I, sig)):
        _same(f, g)


@pytest.mark.parametrize("kind", ["random", "two_by_two", "ties"])
def test_many_shifts_from_memory_equal_the_team(gpu_lib, kind):
    """With 120 shifts of order 2100 the teams do not fit the device until 512 rows are left:
    some 25 panels run from memory, one workgroup a shift, each after the interchanges of
    those before.  One shift alone runs as a team throughout."""
    n = 2100
    A, I = dev(_matrix(kind, n)), dev(np.eye(n))
    sig = [float(s) for s in np.linspace(-31.0, 29.0, 120)]
    facs = gpu_lib.ldlt_factor_multi(A, I, sig)
    for k in (0, 41, 60, 119):
        _same(facs[k], gpu_lib.ldlt_factor(A, I, sig[k]))


def test_captured_factorizations_follow_the_bound(gpu_lib):
    """On a stream of its own a solve replays its captured factorization.  Captured under a
    bound of zero (the sweeps' waits expire), it must not fail the solves that follow."""
    P = inputs.pencil_scf(1200, 120, seed=1)
    A, B = dev(P.A), dev(P.B)
    torch.cuda.synchronize()
    with torch.cuda.stream(torch.cuda.Stream()):
        out = _limited(gpu_lib, 0, lambda: gpu_lib.solve(A, B, 120, 8, check=False))
        assert out["status"] == -2
        for _ in range(3):
            out = gpu_lib.solve(A, B, 120, 8, check=False)
            assert out["status"] == 0
            assert np.max(np.abs(out["evals"].cpu().numpy() - P.lam[:120])) <= 1e-10 * np.max(np.abs(P.lam))
        out = _limited(gpu_lib, 0, lambda: gpu_lib.solve(A, B, 120, 8, check=False))
        assert out["status"] == -2
        out = gpu_lib.solve(A, B, 120, 8, check=False)
        assert out["status"] == 0
    torch.cuda.synchronize()


def _expired_solve(lib):
    """Leaves the word of an expired wait behind an asynchronous solve."""
    n = 1000
    C = inputs.random_symmetric(n, 5)
    f = lib.ldlt_factor(dev(C), dev(np.eye(n)), 0.0)
    Y = dev(np.random.default_rng(1).standard_normal((n, 8)))
    _limited(lib, 0, lambda: lib.ldlt_solve(f, Y))


def _code(call):
    try:
        call()
        return 0
    except SisliceError as e:
        return e.code


def test_expired_wait_is_reported_once_by_the_next_synchronising_call(gpu_lib):
    """By the first factorization that is read back, before its counts are used, and whatever
    else would have ended the call; the call after it starts with a clear word."""
    P = inputs.pencil_scf(600, 60, seed=1)
    A, B = dev(P.A), dev(P.B)
    bad = B.clone()
    bad[100, 100] = -1.0
    calls = [lambda: gpu_lib.plan_shifts_kpm(A, B, 60, 4), lambda: gpu_lib.solve(A, B, 60, 4),
             lambda: gpu_lib.ldlt_factor(A, B, 0.1), lambda: gpu_lib.solve(A, bad, 60, 4)]
    after = [0, 0, 0, -1]   # B is not positive definite
    for call, st in zip(calls, after):
        _expired_solve(gpu_lib)
        assert _code(call) == -2
        assert _code(call) == st
        assert _code(call) == st
