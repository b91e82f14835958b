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


# clusters of 9 to 32 vectors that share a block of T, on the mixed path, whose Newton-Schulz steps start above 2e-7: real
# tridiagonal matrices, which the reduction and the back-transformation pass through, so that the vectors come out orthonormal
# but for the rounding of their entries to FP32, 2 x 2^-24 in a product of two of them
@pytest.mark.parametrize("N, k, e", [(48, 9, -46), (48, 16, -45), (64, 32, -46), (96, 24, -47)])
def test_mixed_clusters_to_rounding(N, k, e):
    gu.need_gpu()
    from paper_2312_13051_amd import _lib as L
    n_mat, f4 = 8192, dict(device="cuda")
    g = torch.Generator(device="cuda").manual_seed(N + k)
    d = 0.7 * torch.rand((n_mat, N), generator=g, **f4)
    d[:, :k] = 1.0
    off = 0.01 + 0.05 * torch.rand((n_mat, N - 1), generator=g, **f4)
    off[:, :k - 1] = (1.0 + torch.rand((n_mat, k - 1), generator=g, **f4)) * 2.0 ** e
    off[:, k - 1] = 0.0
    i = torch.arange(N, device="cuda")
    H = torch.zeros((n_mat, N, N), dtype=torch.complex64, device="cuda")
    H[:, i, i], H[:, i[:-1], i[1:]], H[:, i[1:], i[:-1]] = (x.to(torch.complex64) for x in (d, off, off))
    U = gu.colmajor(n_mat, N, k, N, fill=0)
    ev = torch.empty((n_mat, k + 2), dtype=torch.float64, device="cuda")
    st = torch.empty(n_mat, dtype=torch.int32, device="cuda")
    c = gu.ctx()
    try:
        c.eigh_batched(H, L.BE_C64, N, N, H.stride(0), n_mat, N - k, N, L.BE_MIXED_FP32, ev, U, N, U.stride(0), st)
    finally:
        c.close()
    X = U.real.contiguous()
    gram = torch.bmm(X, X.transpose(1, 2).contiguous()) - torch.eye(k, dtype=torch.float64, device="cuda")
    assert torch.all(st == 0)
    assert float(gram.abs().max()) <= 1.001 * 2.0 ** -23
