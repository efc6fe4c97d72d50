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


@pytest.mark.parametrize("n", [33, 64, 96, 132])
def test_backward_error_of_plain_elimination(svc, n):
    """The factor's residual A - L L^T is no larger than that of column-by-column
    elimination in float64 (one rounding per operation): blocks, reciprocals and
    the square root's iteration lose nothing.  Root mean square over matrices of
    condition 1e8 to 1e11 whose rows are scaled over six decades."""
    import torch
    say("cholesky residual", n)
    r = np.random.default_rng(n)
    rms = {"plain": 0.0, "gpu": 0.0}
    with svc.Plan(8, 8, 1, (1.0,), (0,), 0) as plan:
        for cond in (8, 9, 10, 11):
            q, _ = np.linalg.qr(r.normal(size=(n, n)))
            s = 10.0 ** r.uniform(-3, 3, n)
            A = (q * 10.0 ** np.linspace(0, -cond, n)) @ q.T * s[:, None] * s[None, :]
            A = (A + A.T) / 2
            P = A.copy()
            for j in range(n):
                P[j, j] = np.sqrt(P[j, j])
                P[j + 1:, j] /= P[j, j]
                P[j + 1:, j + 1:] -= np.outer(P[j + 1:, j], P[j + 1:, j])
            G = to_host(plan.cholesky_factor(torch.from_numpy(A.copy()).cuda()))
            for name, L in (("plain", np.tril(P)), ("gpu", G)):
                L = L.astype(np.longdouble)
                d = np.sqrt(np.diag(A).astype(np.longdouble))
                rms[name] += float(np.mean(((A - L @ L.T) / d[:, None] / d[None, :]) ** 2))
    say("  ", rms)
    assert rms["gpu"] <= rms["plain"]
