"""Small-order eigensolver (one launch per batch, several matrices per wave) against LAPACK at the edges of its lane
groups (orders 8, 16, 32), for batches that do not fill a wave, narrow and full windows and degenerate spectra."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from tests import gpu_util as gu  # noqa: E402

pytestmark = pytest.mark.gpu


def hermitian(n, N, seed, degenerate):
    rng = np.random.default_rng([seed, N])
    A = rng.standard_normal((n, N, N)) + 1j * rng.standard_normal((n, N, N))
    H = A + np.conj(np.swapaxes(A, 1, 2))
    if degenerate:  # levels in threes
        w, V = np.linalg.eigh(H)
        w = np.arange(N)[None] // 3 * 1.5 - 2.0 + 0 * w
        H = (V * w[:, None, :]) @ np.conj(np.swapaxes(V, 1, 2))
        H = 0.5 * (H + np.conj(np.swapaxes(H, 1, 2)))
    return H


# bounds: those of the general solver's tests (FP64: eigenvalues 1e-12 ||H||, orthonormality 2e-11, projector 1e-10 at
# gaps >= 1e-3 ||H||; mixed: 2e-5, 1e-5 and 1e-4, the FP32 reduction's)
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("degenerate", [False, True])
@pytest.mark.parametrize("N, lo, hi, n", [(1, 0, 1, 5), (2, 0, 1, 9), (4, 0, 2, 17), (8, 3, 8, 7), (9, 0, 9, 6), (16, 6, 10, 5),
                                          (17, 0, 8, 3), (31, 9, 30, 2), (32, 0, 32, 3), (32, 15, 15, 2), (33, 0, 16, 2),
                                          (64, 0, 32, 2), (65, 3, 60, 2)])
def test_small_orders(N, lo, hi, n, degenerate, precision):
    gu.need_gpu()
    from paper_2312_13051_amd import _lib as L
    H = hermitian(n, N, 3, degenerate)
    m, ld = hi - lo, N + 1
    mixed = precision == "mixed"
    bound = (2e-5, 1e-5, 1e-4) if mixed else (1e-12, 2e-11, 1e-10)
    c = gu.ctx()
    try:
        dH = gu.from_np(np.tril(H) + np.triu(np.full((N, N), 7.0), 1), ld, torch.complex64 if mixed else torch.complex128)
        U = gu.colmajor(n, N, max(m, 1), N + 2, fill=0)
        ev = torch.empty((n, m + 2), dtype=torch.float64, device="cuda")
        st = torch.full((n,), 77, dtype=torch.int32, device="cuda")
        c.eigh_batched(dH, L.BE_C64 if mixed else L.BE_C128, N, ld, dH.stride(0), n, lo, hi,
                       L.BE_MIXED_FP32 if mixed else L.BE_FP64, ev, U, N + 2, U.stride(0), st)
        ev, U, st = ev.cpu().numpy(), gu.to_np(U, N)[:, :, :m], st.cpu().numpy()
    finally:
        c.close()
    for q in range(n):
        w, V = np.linalg.eigh(H[q])
        nrm = max(1.0, np.abs(w).max())
        gaps = [w[k] - w[k - 1] for k in (lo, hi) if m and 0 < k < N]
        if not mixed:
            assert st[q] == (1 if gaps and min(gaps) < 1e-9 * nrm else 0)
        assert np.abs(ev[q, 1:m + 1] - w[lo:hi]).max(initial=0.0) <= bound[0] * nrm
        assert (ev[q, 0] == ev[q, 0]) == (lo > 0) and (ev[q, m + 1] == ev[q, m + 1]) == (hi < N)
        assert np.abs(U[q].conj().T @ U[q] - np.eye(m)).max(initial=0.0) < bound[1]
        if m and (not gaps or min(gaps) > 1e-3 * nrm):
            P = U[q] @ U[q].conj().T - V[:, lo:hi] @ V[:, lo:hi].conj().T
            assert np.abs(P).max() < bound[2] * (1 if not gaps else max(1.0, 0.05 * nrm / min(gaps)))


# every order of the one-launch mixed solve and the next, whole window on the refined path (FP64 subspace: its tests' bounds)
@pytest.mark.parametrize("precision", ["mixed", "refined"])
@pytest.mark.parametrize("N", range(1, 18))
def test_mixed_orders(N, precision):
    gu.need_gpu()
    from paper_2312_13051_amd import _lib as L
    H, n, mixed = hermitian(9, N, 6, N % 2 == 0), 9, precision == "mixed"
    lo, hi = (0, N) if mixed else (N // 4, N)
    m, bound = hi - lo, 1e-5 if mixed else 1e-12
    c = gu.ctx()
    try:
        dH = gu.from_np(H, N + 2, torch.complex64 if mixed else torch.complex128)
        U = gu.colmajor(n, N, m, N + 1, fill=0)
        ev = torch.empty((n, m + 2), dtype=torch.float64, device="cuda")
        st = torch.full((n,), 77, dtype=torch.int32, device="cuda")
        c.eigh_batched(dH, L.BE_C64 if mixed else L.BE_C128, N, N + 2, dH.stride(0), n, lo, hi,
                       L.BE_MIXED_FP32 if mixed else L.BE_MIXED_FP32_REFINED, ev, U, N + 1, U.stride(0), st)
        ev, U = ev.cpu().numpy(), gu.to_np(U, N)[:, :, :m]
    finally:
        c.close()
    for q in range(n):
        w = np.linalg.eigvalsh(H[q])
        nrm = max(1.0, np.abs(w).max())
        assert np.abs(ev[q, 1:m + 1] - w[lo:hi]).max() <= 2e-5 * nrm
        assert np.abs(U[q].conj().T @ U[q] - np.eye(m)).max() < bound
        if mixed:
            assert np.abs(H[q] @ U[q] - U[q] * ev[q, 1:m + 1]).max() <= 1e-4 * nrm


# the flags of every small solver (FP64, the one-launch mixed one, the tridiagonal part alone from 17 on, the refined path on
# either): none for separated levels, a closed gap where all levels are one, non-finite input flagged with NaN levels, and no
# matrix touched by its neighbours' flags
@pytest.mark.parametrize("precision", ["fp64", "mixed", "refined"])
@pytest.mark.parametrize("N", [2, 4, 5, 8, 9, 15, 16, 17, 24, 32, 33])
def test_status(N, precision):
    gu.need_gpu()
    from paper_2312_13051_amd import _lib as L
    mixed, n, (lo, hi) = precision == "mixed", 9, (N // 4, N // 2 + (N > 2))
    m = hi - lo
    rng = np.random.default_rng([N, 11])
    H = np.empty((n, N, N), complex)
    for q in range(n):  # levels 1, 2, 3, ...
        Q = np.linalg.qr(rng.standard_normal((N, N)) + 1j * rng.standard_normal((N, N)))[0]
        H[q] = (Q * np.arange(1.0, N + 1)) @ Q.conj().T
    H = 0.5 * (H + H.conj().transpose(0, 2, 1))
    want = np.zeros(n, int)
    for q, v in ((2, np.nan), (5, np.inf)):
        H[q, N - 1, 0] = v
        want[q] = L.ST_NAN_INF
    H[7] = 1.5 * np.eye(N)
    want[7] = L.ST_GAP_CLOSED
    c = gu.ctx()
    try:
        dH = gu.from_np(H, N, torch.complex64 if mixed else torch.complex128)
        U = gu.colmajor(n, N, m, N, fill=0)
        ev = torch.empty((n, m + 2), dtype=torch.float64, device="cuda")
        st = torch.full((n,), 77, dtype=torch.int32, device="cuda")
        c.eigh_batched(dH, L.BE_C64 if mixed else L.BE_C128, N, N, dH.stride(0), n, lo, hi,
                       {"fp64": L.BE_FP64, "mixed": L.BE_MIXED_FP32, "refined": L.BE_MIXED_FP32_REFINED}[precision], ev, U, N,
                       U.stride(0), st)
        ev, st = ev.cpu().numpy(), st.cpu().numpy()
    finally:
        c.close()
    bad = want == L.ST_NAN_INF
    assert np.array_equal(st[~bad], want[~bad]) and np.all(st[bad] & L.ST_NAN_INF)
    assert np.all(np.isnan(ev[bad, 1:m + 1]))
    good = ev[want == 0, 1:m + 1]
    assert np.abs(good - np.arange(lo + 1, hi + 1)).max() <= (2e-5 if mixed else 1e-10) * N
