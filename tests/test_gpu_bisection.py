"""Sturm counts by principal minors: orders around the counts' groups of eight rows, matrices that split, are scaled far
from one or graded over many decades, against LAPACK."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from tests import gpu_util as gu  # noqa: E402
from tests.test_gpu_eigh import run_eigh  # noqa: E402

pytestmark = pytest.mark.gpu


def tridiagonal(N, kind, rng):
    d, e = rng.standard_normal(N), rng.standard_normal(N - 1)
    if kind == "split":  # repeated diagonal blocks with zero couplings, a zero level among them
        d, e = np.resize([1.0, -1.0, 0.0], N), np.where(np.arange(1, N) % 3 == 0, 0.0, 0.5)
    elif kind == "graded":
        g = 10.0 ** -np.linspace(0.0, 30.0, N)
        d, e = d * g, e * np.sqrt(g[1:] * g[:-1])
    return np.diag(d) + np.diag(e, -1) + np.diag(e, 1)


# bound: backward stability, N eps ||H|| for each of reduction, counts and LAPACK's own
@pytest.mark.parametrize("scale", [1.0, 2.0 ** -400, 2.0 ** 400])
@pytest.mark.parametrize("kind", ["random", "split", "graded"])
@pytest.mark.parametrize("N", [2, 8, 9, 10, 17, 32, 40, 41, 42, 48, 300])
def test_eigenvalues(N, kind, scale):
    gu.need_gpu()
    H = tridiagonal(N, kind, np.random.default_rng([N, 5])).astype(complex)[None]
    c = gu.ctx()
    try:
        ev = run_eigh(c, H * scale, 0, N)[0]
    finally:
        c.close()
    w = np.linalg.eigvalsh(H[0])
    assert np.abs(ev[0, 1:-1] / scale - w).max() <= 3 * N * np.finfo(float).eps * np.abs(w).max()
