"""Orthonormalization of large clusters (panels of 16 vectors on the matrix cores): degenerate levels at the edges of the
panels and of the row tiles, two clusters in a matrix, clusters spread below the cluster tolerance, against LAPACK."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from tests import gpu_util as gu  # noqa: E402
from tests.test_gpu_eigh import check, run_eigh  # noqa: E402

pytestmark = pytest.mark.gpu


# bounds: those of the general solver's tests (projector and residual of the window, orthonormality 2e-11)
@pytest.mark.parametrize("spread", [0.0, 1e-14])
@pytest.mark.parametrize("N, k", [(70, 17), (70, 32), (70, 33), (97, 47), (97, 48), (100, 49), (130, 64), (131, 65), (200, 100),
                                  (333, 150)])
def test_large_clusters(N, k, spread):
    gu.need_gpu()
    rng = np.random.default_rng([N, k])
    Hs = []
    for rest in (rng.uniform(2.0, 3.0, N - k), np.full(N - k, 1.0)):
        Q = np.linalg.qr(rng.standard_normal((N, N)) + 1j * rng.standard_normal((N, N)))[0]
        H = (Q * np.concatenate([-1.0 + spread * rng.standard_normal(k), rest])) @ Q.conj().T
        Hs.append(0.5 * (H + H.conj().T))
    Hs = np.stack(Hs)
    c = gu.ctx()
    try:
        check(Hs, 0, k, *run_eigh(c, Hs, 0, k))
        check(Hs, 0, N, *run_eigh(c, Hs, 0, N))
    finally:
        c.close()
