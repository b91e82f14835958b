"""Bloch Hamiltonians with the phases of the distinct lattice vectors in LDS: against the oracle, and bit for bit against
the path without the table, which longer vector lists take."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import synthetic as syn  # noqa: E402
from oracle import berry as orc  # noqa: E402
from tests import gpu_util as gu  # noqa: E402

pytestmark = pytest.mark.gpu


def chain_of_vectors(N, n_R, seed, extra=()):
    """N orbitals, 2 n_R + 1 distinct vectors (0 and +-R), every vector in several orbital pairs; extra vectors get a zero
    amplitude."""
    rng = np.random.default_rng([seed, N])
    blocks = {(0, 0): np.diag(rng.standard_normal(N)).astype(complex)}
    for r in range(n_R):
        T = np.zeros((N, N), dtype=complex)
        for _ in range(2 * N):
            T[rng.integers(N), rng.integers(N)] = complex(*rng.standard_normal(2))
        blocks[(1 + r % 7, r // 7 - 3)] = T
    i, j, R, t = [], [], [], []
    for v, T in blocks.items():
        for s in ((1, -1) if any(v) else (1,)):
            a, b = np.nonzero(T)
            i.append(a if s == 1 else b)
            j.append(b if s == 1 else a)
            R.append(np.tile(np.array(v) * s, (a.size, 1)))
            t.append(T[a, b] if s == 1 else T[a, b].conj())
    for v in extra:
        for s in (1, -1):
            i.append([0]), j.append([0]), R.append(np.array([v]) * s), t.append([0j])
    return syn.HopList(N, 2, np.concatenate(i).astype(np.int32), np.concatenate(j).astype(np.int32),
                       np.concatenate(R).astype(np.int32), np.concatenate(t))


def build(ctx, hops, kappa, dtype, pad):
    from paper_2312_13051_amd import _lib as L
    N = hops[0].N
    plan = ctx.hk_plan(hops)
    n = len(hops) * len(kappa)
    H = gu.colmajor(n, N, N, N + pad, torch.complex128 if dtype == L.BE_C128 else torch.complex64, fill=3)
    ctx.build_hk(plan, 0, len(hops), torch.from_numpy(kappa).cuda(), H, H.stride(0), N + pad, dtype)
    return H.cpu().numpy()[:, :, :N].swapaxes(1, 2)


# lanes per matrix 8 .. 256 with the table full (2,048 phases over the workgroup's matrices) and overfull by one pair of
# vectors, which takes the path without it; matrices that do not fill a workgroup, systems of different lists; k-points
# four at a time (511 vectors are the most that still fit so) and one at a time
@pytest.mark.parametrize("N, n_R, n_k", [(2, 31, 33), (3, 5, 1), (5, 60, 7), (20, 9, 3), (40, 100, 2),
                                         (40, 255, 9), (40, 256, 5)])
@pytest.mark.parametrize("dtype", [0, 1])
def test_phase_table(N, n_R, n_k, dtype):
    gu.need_gpu()
    kappa = np.random.default_rng(N).uniform(-1, 1, (n_k, 3))
    hops = [chain_of_vectors(N, n_R, s) for s in range(2)]
    more = [chain_of_vectors(N, n_R, s, extra=[(20 + e, 40) for e in range(1100)]) for s in range(2)]
    c = gu.ctx()
    try:
        H, H2 = build(c, hops, kappa, dtype, 3), build(c, more, kappa, dtype, 0)
    finally:
        c.close()
    assert np.array_equal(H, H2)
    ref = np.stack([orc.bloch_hamiltonian(h, k) for h in hops for k in kappa])
    # at most 2 n_R + 1 terms an element, each with a phase argument up to ~20 turns: 20 (2 n_R + 1) eps max|t|
    scale = max(np.abs(h.t).max() for h in hops)
    eps = 2.3e-16 if dtype == 0 else 6e-8
    assert np.abs(H - ref).max() < 20 * (2 * n_R + 1) * eps * scale
    assert np.array_equal(H, np.conj(H.swapaxes(1, 2)))


# lists around the share of pairs from which the others are filled in (half, and eight more), alone and beside a sparse one:
# every element of H is written
@pytest.mark.parametrize("N, share", [(1, 0.0), (2, 0.3), (4, 0.2), (4, 0.6), (9, 0.3), (9, 0.45), (9, 0.9), (40, 0.4), (40, 0.6)])
@pytest.mark.parametrize("dtype", [0, 1])
def test_every_element_written(N, share, dtype):
    gu.need_gpu()
    rng = np.random.default_rng([N, int(100 * share)])
    hops = []
    for sh in (share, 0.1):
        a, b = np.nonzero(np.triu(rng.random((N, N)) < sh))
        t = rng.standard_normal(a.size) + 1j * np.where(a == b, 0.0, rng.standard_normal(a.size))
        off = a != b
        i, j = np.concatenate([a, b[off]]), np.concatenate([b, a[off]])
        hops.append(syn.HopList(N, 2, i.astype(np.int32), j.astype(np.int32), np.zeros((i.size, 2), np.int32),
                                np.concatenate([t, t[off].conj()])))
    kappa = rng.uniform(-1, 1, (5, 3))
    c = gu.ctx()
    try:
        for hs in (hops[:1], hops):
            H = build(c, hs, kappa, dtype, 2)
            ref = np.zeros((len(hs), N, N), complex)
            for s, h in enumerate(hs):
                ref[s, h.i, h.j] = h.t
            assert np.abs(H - np.repeat(ref, 5, axis=0)).max(initial=0.0) <= (0.0 if dtype == 0 else 1e-6)
    finally:
        c.close()


# the number of k-points decides how many share an entry's read and how many pairs a workgroup takes: the same bits for each
# k-point alone, a few at a time and all together, with few entries a pair and many
@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("model", ["sparse", "dense"])
def test_same_bits_in_any_call(model, dtype):
    gu.need_gpu()
    hop = syn.bhz_disordered(16, 1.0, [3, 5]) if model == "sparse" else syn.wannier_like(40, [3, 6])
    kappa = np.random.default_rng(7).uniform(-1, 1, (110, 3))
    c = gu.ctx()
    try:
        H = build(c, [hop], kappa, dtype, 0)
        for part in (slice(3, 4), slice(10, 17), slice(40, 105)):
            assert np.array_equal(build(c, [hop], kappa[part], dtype, 0), H[part])
    finally:
        c.close()
