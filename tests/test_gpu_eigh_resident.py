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
