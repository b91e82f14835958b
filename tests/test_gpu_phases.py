"""Eigenphases of Wilson matrices with chosen spectra: the QR (orders up to 12) and the Hermitian problem (from 13 on, in LDS
up to 32), with phases placed against the latter: pairs on both sides of its branch point and crowds of equal ones."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from tests import gpu_util as gu  # noqa: E402
from tests.phase_metrics import phase_set_error  # noqa: E402

pytestmark = pytest.mark.gpu

PHI = 0.6180339887498949  # the shift of (e^{-i phi} W + e^{i phi} W^H) / 2


def grid_with_phases(theta, seed):
    """A closed line of three points whose Wilson matrix has the given phases (|theta| < pi/2): in a common random basis,
    point j holds the two-component vectors (1, 0), (1, 1)/sqrt 2, (1, e^{-2 i theta})/sqrt 2 of each band."""
    m = theta.size
    rng = np.random.default_rng(seed)
    V = np.linalg.qr(rng.standard_normal((m, m)) + 1j * rng.standard_normal((m, m)))[0]
    r = np.sqrt(0.5)
    parts = [(np.ones(m), np.zeros(m)), (r * np.ones(m), r * np.ones(m)), (r * np.ones(m), r * np.exp(-2j * theta))]
    return np.stack([np.concatenate([(V * a) @ V.conj().T, (V * b) @ V.conj().T]) for a, b in parts])


# phases by |theta| up to 1.4; acos loses eps / |sin| >= 0.005, on matrices unitary to ~100 eps: 100 * 2.2e-16 / 0.005 = 4e-12
@pytest.mark.parametrize("m", [12, 13, 16, 17, 32, 33, 64, 100, 101])
@pytest.mark.parametrize("kind", ["spread", "pairs", "crowd"])
def test_chosen_phases(m, kind):
    gu.need_gpu()
    lines = []
    rng = np.random.default_rng([m, len(kind)])
    for _ in range(3):
        th = rng.uniform(-1.4, 1.4, m)
        if kind == "pairs":  # theta - phi = +-x, the cosines equal to within 1e-7 .. 1e-12, x down to the branch point
            x = np.array([0.3, 0.04, 0.01, 0.002])
            th[:4] = PHI + x
            th[4:8] = PHI - x * (1.0 + np.array([1e-7, 1e-6, 1e-5, 1e-8]))
        elif kind == "crowd":
            th[:m // 2] = 0.25 + 1e-11 * rng.standard_normal(m // 2)
        lines.append(th)
    U = np.stack([grid_with_phases(th, [m, q]) for q, th in enumerate(lines)])
    c = gu.ctx()
    try:
        Ud = gu.from_np(U.reshape(-1, 2 * m, m), 2 * m)
        f8 = dict(dtype=torch.float64, device="cuda")
        i4 = dict(dtype=torch.int32, device="cuda")
        out, phi = torch.empty((1, 3, m), **f8), torch.empty((1, 3), **f8)
        wn, st = torch.empty(1, **i4), torch.empty(1, **i4)
        c.wilson_loop(Ud, 2 * m, m, 2 * m, Ud.stride(0), 1, 3, 3, 0, out, phi, wn, st)
        got, status = out[0].cpu().numpy(), int(st[0])
    finally:
        c.close()
    assert status & ~4 == 0
    assert phase_set_error(got, np.array(lines)) < 4e-12
    assert np.all(np.diff(got, axis=1) >= 0)


# orders whose Hermitian problems, few of them, are reduced by column launches before the on-chip reduction takes the last
# columns: one panel, a panel and one column more, blocks of 64 rows with remainders
@pytest.mark.parametrize("m", [217, 248, 249, 300, 513])
@pytest.mark.parametrize("kind", ["spread", "crowd"])
def test_few_large_orders(m, kind):
    test_chosen_phases(m, kind)


def round_loop(theta, n_par, seed):
    """A closed line of n_par points whose Wilson matrix has the given phases: in a common random basis, each band's two
    components go round a circle, (sqrt(1 - p), sqrt(p) e^{i delta j}), delta = 2 pi / n_par, with the p whose links have the
    phase theta / n_par. All links are well conditioned (singular values from cos(pi / n_par) up)."""
    m = theta.size
    rng = np.random.default_rng(seed)
    V = np.linalg.qr(rng.standard_normal((m, m)) + 1j * rng.standard_normal((m, m)))[0]
    delta = 2 * np.pi / n_par
    t = np.tan(np.abs(theta) / n_par)
    p = t / (np.sin(delta) + t * (1 - np.cos(delta)))
    return np.stack([np.concatenate([(V * np.sqrt(1 - p)) @ V.conj().T,
                                     (V * (np.sqrt(p) * np.exp(-1j * np.sign(theta) * delta * j))) @ V.conj().T])
                     for j in range(n_par)])


# phases 0.05 to 0.06 from the branch point of the Hermitian problem, on either side, where a phase from the cosine alone is off
# by eps / |sin| and the cosine's own errors, and well-separated ones: as near as the matrices are unitary, to about 100 eps
@pytest.mark.parametrize("m", [12, 13, 16, 33, 48, 64, 100])
@pytest.mark.parametrize("kind", ["near", "spread"])
def test_phases_to_rounding(m, kind):
    gu.need_gpu()
    rng = np.random.default_rng([m, len(kind), 5])
    lines = []
    for _ in range(8):
        th = rng.uniform(-1.4, 1.4, m)
        if kind == "near":
            th[:m // 2] = PHI + rng.choice([-1.0, 1.0], m // 2) * rng.uniform(0.05, 0.06, m // 2)
        lines.append(th)
    got, status = loop_phases(np.stack([round_loop(th, 16, [m, q, 5]) for q, th in enumerate(lines)]))
    assert status & ~4 == 0
    assert phase_set_error(got, np.array(lines)) < 100 * np.finfo(float).eps


def loop_phases(U):
    """Phases and status of one system's Wilson loops over the lines of U (line, point, N, m)."""
    n_perp, n_par, N, m = U.shape
    f8 = dict(dtype=torch.float64, device="cuda")
    i4 = dict(dtype=torch.int32, device="cuda")
    c = gu.ctx()
    try:
        Ud = gu.from_np(U.reshape(-1, N, m), N)
        out, phi = torch.empty((1, n_perp, m), **f8), torch.empty((1, n_perp), **f8)
        wn, st = torch.empty(1, **i4), torch.empty(1, **i4)
        c.wilson_loop(Ud, N, m, N, Ud.stride(0), 1, n_par, n_perp, 0, out, phi, wn, st)
        return out[0].cpu().numpy(), int(st[0])
    finally:
        c.close()


def newton_schulz(F):
    """The polar iteration of the loops' links: at most 51 steps of X (3 I - X^H X) / 2."""
    eye = np.eye(F.shape[0])
    for _ in range(51):
        G = F.conj().T @ F
        err = np.abs(G - eye).max()
        F = F @ (1.5 * eye - 0.5 * G)
        if err < 1e-7:
            break
    return F


# a link with a singular value that 51 steps take to 0.45, 0.9995 or 0.99994: the line is flagged, its W is neither unitary
# nor normal, and its phases are the arguments of W's eigenvalues. The value is uncertain by the rounding of the link's
# entries, 2 m eps relative to the value at the start, and the phases with it
@pytest.mark.parametrize("m", [12, 13, 48, 100, 101])
@pytest.mark.parametrize("smin", [5e-10, 3e-9, 3.5e-9])
def test_link_not_converged(m, smin):
    gu.need_gpu()
    rng = np.random.default_rng([m, 6])
    P, Q, P2, Q2 = (np.linalg.qr(rng.standard_normal((m, m)) + 1j * rng.standard_normal((m, m)))[0] for _ in range(4))
    s = np.r_[smin, np.ones(m - 1)]
    U = np.stack([np.concatenate([np.eye(m), np.zeros((m, m))]),
                  np.concatenate([(P * s) @ Q.conj().T, (Q * np.sqrt(1 - s * s)) @ Q.conj().T]),
                  np.concatenate([0.8 * P2 @ Q2.conj().T, 0.6 * np.eye(m)])])[None]
    F = [newton_schulz(U[0, (j + 1) % 3].conj().T @ U[0, j]) for j in range(3)]
    got, status = loop_phases(U)
    assert status & 2
    assert phase_set_error(got, np.angle(np.linalg.eigvals(F[2] @ F[1] @ F[0]))[None]) < 2 * m * np.finfo(float).eps / smin


def bits(x):
    return x.contiguous().view(torch.int64)


# lines of Wilson matrices above order 216, few enough for column launches (4) and too many for them (100), and line counts on
# either side of the rule (96 on 256 compute units): a system's phases are the same bits alone and in any larger call
@pytest.mark.parametrize("threads", [0, 256, 512, 1024])  # of the panel kernel; 0: the tuning table's
@pytest.mark.parametrize("m,copies", [(217, (25,)), (248, (24, 25)), (249, (25,)), (300, (25,)), (345, (25,)), (513, (25,))])
def test_same_bits_alone_and_in_larger_calls(m, copies, threads):
    gu.need_gpu()
    rng = np.random.default_rng([m, 9])
    lines = np.stack([rng.uniform(-1.2, 1.2, m) for _ in range(4)])
    U = np.stack([grid_with_phases(th, [m, q, 9]) for q, th in enumerate(lines)])
    c = gu.ctx()
    if threads:
        c.tune_clear("hetrd_panel_threads")
        c.tune_set("hetrd_panel_threads", threads)
    try:
        U1 = gu.from_np(U.reshape(-1, 2 * m, m), 2 * m)

        def run(n_sys):
            Ud = U1.repeat(n_sys, 1, 1)
            th, phi = (torch.empty((n_sys, 4) + s, dtype=torch.float64, device="cuda") for s in ((m,), ()))
            wn, st = (torch.empty(n_sys, dtype=torch.int32, device="cuda") for _ in range(2))
            c.wilson_loop(Ud, 2 * m, m, 2 * m, Ud.stride(0), n_sys, 3, 4, 0, th, phi, wn, st)
            torch.cuda.synchronize()
            return th, phi, st
        th, phi, st = run(1)
        assert int(st[0]) & ~4 == 0
        assert phase_set_error(th[0].cpu().numpy(), lines) < 4e-12
        for n in copies:
            th2, phi2, st2 = run(n)
            assert torch.equal(bits(th2), bits(th.repeat(n, 1, 1))) and torch.equal(bits(phi2), bits(phi.repeat(n, 1)))
            assert torch.all(st2 == st)
    finally:
        c.close()


def test_captured_column_launches():
    """A Wilson loop of order 249 (one panel by column launches) under graph capture: every replay equals the eager call."""
    gu.need_gpu()
    m, s = 249, torch.cuda.Stream()
    rng = np.random.default_rng([m, 10])
    U = np.stack([grid_with_phases(rng.uniform(-1.2, 1.2, m), [m, q, 10]) for q in range(3)])
    c = gu.ctx()
    Ud = gu.from_np(U.reshape(-1, 2 * m, m), 2 * m)
    th, phi = torch.empty((1, 3, m), dtype=torch.float64, device="cuda"), torch.empty((1, 3), dtype=torch.float64, device="cuda")
    wn, st = (torch.empty(1, dtype=torch.int32, device="cuda") for _ in range(2))

    def run():
        c.wilson_loop(Ud, 2 * m, m, 2 * m, Ud.stride(0), 1, 3, 3, 0, th, phi, wn, st)
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        run()  # sizes the workspace outside capture
    torch.cuda.synchronize()
    ref = [v.clone() for v in (th, phi, wn, st)]
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s, capture_error_mode="relaxed"):
        run()
    for _ in range(3):
        for v in (th, phi, wn, st):
            v.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip((th, phi, wn, st), ref))
        x = torch.randn(1000, device="cuda")  # eager work between the replays
        assert float(x.abs().sum()) > 0
    c.close()
