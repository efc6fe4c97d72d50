"""Cholesky factor and solve around the 32-column blocks of the kernels."""

import numpy as np
import pytest

from tests.helpers import say, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 31, 32, 33, 64, 65, 97, 294, 1000, 1024])
def test_factor_and_solve(svc, n):
    """A = X^T X with X 3 n x n has condition about 14: the factor's and the
    solution's relative errors are a small multiple of n eps (8 n eps here)."""
    import torch
    r = np.random.default_rng(n)
    X = r.normal(size=(3 * n, n))
    A = X.T @ X
    b = r.normal(size=n)
    say("cholesky", n)
    tol = 8 * n * np.finfo(np.float64).eps
    with svc.Plan(8, 8, 1, (1.0,), (0,), 0) as plan:
        # only the lower triangle is read
        Ad = torch.from_numpy(np.where(np.tril(np.ones((n, n))) > 0, A, np.nan)).cuda()
        plan.cholesky_factor(Ad)
        L, Lref = to_host(Ad), np.linalg.cholesky(A)
        assert np.max(np.abs(L - Lref)) <= tol * np.abs(Lref).max()
        x = to_host(plan.cholesky_solve(Ad, torch.from_numpy(b).cuda()))
    xref = np.linalg.solve(A, b)
    assert np.max(np.abs(x - xref)) <= 4 * tol * np.abs(xref).max()


@pytest.mark.parametrize("n,pivot", [(1, 0), (40, 39), (70, 31), (70, 32), (100, 50)])
def test_pivot_is_reported(svc, n, pivot):
    import torch
    from paper_1209_5823_amd._lib import SvconvError, ENOTSPD
    d = np.ones(n)
    d[pivot] = -1.0
    d[pivot + 1:] = -2.0
    say("cholesky pivot", n, pivot)
    with svc.Plan(8, 8, 1, (1.0,), (0,), 0) as plan:
        with pytest.raises(SvconvError) as ei:
            plan.cholesky_factor(torch.from_numpy(np.diag(d)).cuda())
        assert ei.value.status == ENOTSPD
        assert "pivot %d " % pivot in str(ei.value)
        # the status does not outlive the call
        plan.cholesky_factor(torch.from_numpy(np.eye(n)).cuda())


@pytest.mark.parametrize("n", [1, 3, 6, 16, 31, 32, 33])
def test_one_block_is_written_in_place(svc, n):
    """One launch up to n = 32: the factor below the diagonal, zeros above it, and
    nothing past the matrix."""
    import torch
    r = np.random.default_rng(n)
    X = r.normal(size=(3 * n, n))
    A = X.T @ X
    say("cholesky, one block", n)
    buf = torch.full((n * n + 40,), 7.0, dtype=torch.float64).cuda()
    with svc.Plan(8, 8, 1, (1.0,), (0,), 0) as plan:
        M = buf[:n * n].view(n, n)
        M.copy_(torch.from_numpy(np.where(np.tril(np.ones((n, n))) > 0, A, np.nan)))
        plan.cholesky_factor(M)
        L, Lref = to_host(M), np.linalg.cholesky(A)
    assert np.max(np.abs(L - Lref)) <= 8 * n * np.finfo(np.float64).eps * np.abs(Lref).max()
    assert np.array_equal(np.triu(L, 1), np.zeros((n, n)))
    assert bool((buf[n * n:] == 7.0).all())
