"""Link determinants with a row of the panel per thread: orders around the panels of 16 and the workgroup sizes, links whose
determinant underflows the certificate's first test and links singular to working precision, against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import berry as orc  # noqa: E402
from tests import gpu_util as gu  # noqa: E402
from tests.test_gpu_flux import circ  # noqa: E402

pytestmark = pytest.mark.gpu


# random bases (|det| far below one, the smallest singular value estimated from the factors) and nearby ones; bound: that of
# the flux tests
@pytest.mark.parametrize("near", [False, True])
@pytest.mark.parametrize("m", [1, 2, 15, 16, 17, 31, 63, 64, 65, 127, 128, 129, 192, 255, 256])
def test_orders(m, near):
    gu.need_gpu()
    rng = np.random.default_rng([m, near])
    n_perp, n_par, N = 3, 4, m + 5
    B = rng.standard_normal((n_perp, n_par, N, m)) + 1j * rng.standard_normal((n_perp, n_par, N, m))
    Ug = np.linalg.qr(0.05 * B + B[:1, :1] if near else B)[0]
    if near and m > 1:  # one point's first vector outside the others' span: its links are singular
        Ug[1, 1, :, 0] = 0.0
    U = torch.from_numpy(np.ascontiguousarray(np.swapaxes(Ug, -1, -2).reshape(-1, m, N))).cuda()
    f = torch.empty((n_perp, n_par), dtype=torch.float64, device="cuda")
    ch = torch.empty(1, dtype=torch.int32, device="cuda")
    tot = torch.empty(1, dtype=torch.float64, device="cuda")
    st = torch.empty(1, dtype=torch.int32, device="cuda")
    c = gu.ctx()
    try:
        c.plaquette_flux(U, N, m, N, m * N, 1, n_par, n_perp, f, ch, tot, st)
        f, st = f.cpu().numpy(), int(st[0])
    finally:
        c.close()
    ref = orc.plaquette_flux_from_grid(Ug)
    assert (st & orc.OVERLAP_SINGULAR) == (ref["status"] & orc.OVERLAP_SINGULAR)
    assert bool(st & orc.OVERLAP_SINGULAR) >= (near and m > 1)
    ok = np.ones((n_perp, n_par), bool)
    if near and m > 1:  # plaquettes with a corner at that point have no flux
        ok[np.ix_([0, 1], [0, 1])] = False
    assert circ(f, ref["flux"])[ok].max() < 1e-9


# every panel width at its first and last order, one panel and several with remainders
@pytest.mark.parametrize("near", [False, True])
@pytest.mark.parametrize("m", [3, 4, 5, 8, 9, 12, 13, 59, 60, 61, 66, 79, 80, 81])
def test_panel_widths(m, near):
    test_orders(m, near)
