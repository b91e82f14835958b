"""On-chip Householder reduction (FP64): orders at the edges of its register blocks (64, 96, 128, 160, 192), of its LDS
columns (216) and past them, where the panel kernel takes the first columns, against LAPACK."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from tests import gpu_util as gu  # noqa: E402
from tests.test_gpu_eigh import check, run_eigh  # noqa: E402

pytestmark = pytest.mark.gpu

ORDERS = [33, 64, 65, 96, 97, 128, 129, 160, 161, 192, 193, 200, 215, 216, 217, 248, 249, 288, 331]


@pytest.mark.parametrize("N", ORDERS)
def test_random_orders(N):
    gu.need_gpu()
    rng = np.random.default_rng([N, 1])
    A = rng.standard_normal((3, N, N)) + 1j * rng.standard_normal((3, N, N))
    Hs = A + np.conj(np.swapaxes(A, 1, 2))
    lo, hi = N // 5, N // 5 + N // 2
    c = gu.ctx()
    try:
        check(Hs, lo, hi, *run_eigh(c, Hs, lo, hi))
    finally:
        c.close()


# a spectrum of +-1 (a projected spin operator), a diagonal and an already tridiagonal matrix: reflectors with tau = 0,
# columns of rounding errors, splits of T
@pytest.mark.parametrize("N", [65, 200, 216, 250])
@pytest.mark.parametrize("kind", ["spin", "diagonal", "tridiagonal"])
def test_special_matrices(N, kind):
    gu.need_gpu()
    rng = np.random.default_rng([N, 2])
    if kind == "spin":
        Q = np.linalg.qr(rng.standard_normal((N, N)) + 1j * rng.standard_normal((N, N)))[0]
        H = (Q * np.where(np.arange(N) < N // 3, -1.0, 1.0)) @ Q.conj().T
    elif kind == "diagonal":
        H = np.diag(rng.standard_normal(N)).astype(complex)
    else:
        e = rng.standard_normal(N - 1) + 1j * rng.standard_normal(N - 1)
        H = np.diag(rng.standard_normal(N)).astype(complex) + np.diag(e, -1) + np.diag(e.conj(), 1)
    Hs = 0.5 * (H + H.conj().T)[None]
    c = gu.ctx()
    try:
        check(Hs, 0, N, *run_eigh(c, Hs, 0, N))
    finally:
        c.close()


def scaled_errors(c, H, scale):
    """Largest eigenvalue, orthonormality and residual errors of a full solve of H * scale, relative to the norm."""
    N = H.shape[0]
    ev, U, st = run_eigh(c, (H * scale)[None], 0, N)
    w, lam, nrm = np.linalg.eigvalsh(H), ev[0, 1:-1] / scale, np.abs(H).sum(1).max()
    assert st[0] == 0
    return (np.abs(lam - w).max() / nrm, np.abs(U[0].conj().T @ U[0] - np.eye(N)).max(),
            np.abs(H @ U[0] - U[0] * lam).max() / nrm)


# dense matrices far from norm one (powers of two: the same matrix to the last bit), bounds of the general solver's tests
@pytest.mark.parametrize("scale", [2.0 ** -400, 2.0 ** 400])
@pytest.mark.parametrize("N", [32, 33, 64, 200, 216, 250])
def test_scaled_dense_matrices(N, scale):
    gu.need_gpu()
    rng = np.random.default_rng([N, 3])
    A = rng.standard_normal((N, N)) + 1j * rng.standard_normal((N, N))
    c = gu.ctx()
    try:
        errors = scaled_errors(c, A + A.conj().T, scale)
    finally:
        c.close()
    assert errors[0] <= 1e-12 and errors[1] < 2e-11 and errors[2] < 1e-11


# a first column whose entries' squares leave the range of FP64 (below 1e-154 they are subnormal, below 1e-162 zero)
@pytest.mark.parametrize("tiny", [1e-150, 1e-158, 1e-161, 1e-170])
@pytest.mark.parametrize("N", [33, 100, 216])
def test_column_of_tiny_entries(N, tiny):
    gu.need_gpu()
    rng = np.random.default_rng([N, 4])
    A = rng.standard_normal((N, N)) + 1j * rng.standard_normal((N, N))
    A = A + A.conj().T
    A[1:, 0] *= tiny
    A[0, 1:] = A[1:, 0].conj()
    c = gu.ctx()
    try:
        errors = scaled_errors(c, A, 1.0)
    finally:
        c.close()
    assert errors[0] <= 1e-12 and errors[1] < 2e-11 and errors[2] < 1e-11
