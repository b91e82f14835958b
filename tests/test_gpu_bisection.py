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


# levels far below the norm whose rows couple to the rest by nothing, and among themselves by less than the rounding of the
# norm. The reduction passes these real tridiagonal matrices through, so each block's levels are found to the block's own
# backward error or to the bisection's floor, eps^2 ||H||
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("N", [4, 8, 9, 16, 17, 32, 40, 300])
def test_levels_of_decoupled_blocks(N, precision):
    gu.need_gpu()
    from paper_2312_13051_amd import _lib as L
    mixed, n1 = precision == "mixed", N // 2
    rng = np.random.default_rng([N, 8])
    blocks = [tridiagonal(n, "random", rng).astype(np.float32).astype(float) for n in (n1, N - n1)]
    small = 2.0 ** -66
    H = np.zeros((N, N))
    H[:n1, :n1], H[n1:, n1:] = blocks[0], blocks[1] * small
    c = gu.ctx()
    try:
        dH = gu.from_np(H.astype(complex)[None], N, torch.complex64 if mixed else torch.complex128)
        U = gu.colmajor(1, N, N, N, fill=0)
        ev = torch.empty((1, N + 2), dtype=torch.float64, device="cuda")
        st = torch.empty(1, dtype=torch.int32, device="cuda")
        c.eigh_batched(dH, L.BE_C64 if mixed else L.BE_C128, N, N, dH.stride(0), 1, 0, N,
                       L.BE_MIXED_FP32 if mixed else L.BE_FP64, ev, U, N, U.stride(0), st)
        got = ev[0, 1:-1].cpu().numpy()
    finally:
        c.close()
    eps = np.finfo(float).eps
    w1, w2 = (np.linalg.eigvalsh(b) for b in blocks)
    n0 = int((w1 < 0).sum())
    near, far = got[n0:n0 + w2.size], np.concatenate([got[:n0], got[n0 + w2.size:]])
    assert np.abs(far - w1).max() <= 3 * N * eps * np.abs(w1).max()
    assert np.abs(near - w2 * small).max() <= 3 * N * eps * np.abs(w2).max() * small + 4 * eps ** 2 * np.abs(w1).max()


# uncoupled chains of three sites, one zero level each: the same value for all of them, bit for bit (the bisection of each sees
# the same counts), as the refined path's correction, which divides by differences of levels and skips those of zero, needs
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("N", [6, 9, 15, 18, 33, 60, 300])
def test_equal_levels_of_decoupled_blocks(N, precision):
    gu.need_gpu()
    from paper_2312_13051_amd import _lib as L
    mixed = precision == "mixed"
    e = np.where(np.arange(1, N) % 3 == 0, 0.0, 0.75)
    H = (np.diag(e, 1) + np.diag(e, -1)).astype(complex)[None]
    c = gu.ctx()
    try:
        dH = gu.from_np(H, N, torch.complex64 if mixed else torch.complex128)
        U = gu.colmajor(1, N, N, N, fill=0)
        ev = torch.empty((1, N + 2), dtype=torch.float64, device="cuda")
        st = torch.empty(1, dtype=torch.int32, device="cuda")
        c.eigh_batched(dH, L.BE_C64 if mixed else L.BE_C128, N, N, dH.stride(0), 1, 0, N,
                       L.BE_MIXED_FP32 if mixed else L.BE_FP64, ev, U, N, U.stride(0), st)
        zero = ev[0, 1 + N // 3:1 + 2 * (N // 3)].cpu().numpy()
    finally:
        c.close()
    assert np.abs(zero).max() <= 4 * np.finfo(float).eps ** 2
    assert np.all(zero == zero[0])


# a window that cuts the pair of zero levels of a ring of four sites: flagged for its gap, and a basis all the same
@pytest.mark.parametrize("lo,hi", [(0, 2), (1, 2), (2, 4)])
def test_refined_window_through_equal_levels(lo, hi):
    gu.need_gpu()
    from paper_2312_13051_amd import _lib as L
    P = np.roll(np.eye(4), 1, 0)
    m = hi - lo
    c = gu.ctx()
    try:
        dH = gu.from_np((P + P.T).astype(complex)[None], 4)
        U = gu.colmajor(1, 4, m, 4, fill=0)
        ev = torch.empty((1, m + 2), dtype=torch.float64, device="cuda")
        st = torch.empty(1, dtype=torch.int32, device="cuda")
        c.eigh_batched(dH, L.BE_C128, 4, 4, dH.stride(0), 1, lo, hi, L.BE_MIXED_FP32_REFINED, ev, U, 4, U.stride(0), st)
        V, status, w = U[0].cpu().numpy().T, int(st[0]), ev[0, 1:-1].cpu().numpy()
    finally:
        c.close()
    assert status == L.ST_GAP_CLOSED
    assert np.abs(V.conj().T @ V - np.eye(m)).max() < 1e-13
    assert np.abs(w - np.array([-2.0, 0.0, 0.0, 2.0])[lo:hi]).max() < 1e-12
