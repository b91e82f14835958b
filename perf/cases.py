"""Timed cases of the Wilson-loop engine, through its public Python calls.

A case is a tight-binding model on a k-plane and one of the paper's
calculations on it: the hybrid Wannier centres (``wilson``), the nested loop
(``nested``), the spin-resolved loop (``spin``) or the Berry flux per plaquette
of the occupied space (``flux``) or of its spin sectors (``spin_flux``).
Every pass builds the Bloch Hamiltonians, diagonalizes them and runs the loop
stage. Half filling throughout.

Outputs are the gauge-invariant results: phases, windings, fluxes, projected
spin spectra, eigenvalues, status words. The eigenvectors themselves are left
out: each is defined up to a phase only, and inside a degenerate level up to a
rotation.

The models are those of the repository's workloads (two-band Chern insulator,
BHZ and BBH and their 3D relative, supercells with vacancies and disorder, a
random many-orbital stand-in for a Wannier90 model), written here from a seed.
Grids start at a random offset: on the symmetric lines of the zone the phases
of these models sit exactly on the branch cut at pi, where the sign of a
rounding error decides. For the same reason the four-band models carry a small
random on-site term where nothing else breaks their symmetries.
"""
import math
from dataclasses import dataclass

import numpy as np
import torch

from paper_2312_13051_amd import _lib, pipeline

S0 = np.eye(2, dtype=np.complex128)
S1 = np.array([[0, 1], [1, 0]], dtype=np.complex128)
S2 = np.array([[0, -1j], [1j, 0]], dtype=np.complex128)
S3 = np.array([[1, 0], [0, -1]], dtype=np.complex128)
PRECISION = {"fp64": _lib.BE_FP64, "mixed": _lib.BE_MIXED_FP32, "refined": _lib.BE_MIXED_FP32_REFINED}
ORBITALS = {"qwz": 2, "bhz": 4, "bbh": 4, "choti": 4}  # per site; "wannier": the case's L
SPIN_BHZ = np.array([1.0, -1.0, -1.0, 1.0])  # spin of the orbitals of a BHZ site


def case(name, call, model, L, vacancies, disorder, systems, n_perp, n_par, precision, whole=False):
    """systems: disorder realizations, or parallel planes of the 3D model.
    whole: the pass starts from the hopping lists, as a script does that
    handles each model once; else from the packed plan a program keeps."""
    d = dict(call=call, model=model, L=L, vacancies=vacancies, disorder=disorder, systems=systems, n_perp=n_perp,
             n_par=n_par, precision=precision, whole=whole)
    return dict(d, name=name) if name else d


def listed():
    return [
        # the paper's first example, a two-band Chern insulator on a 64 x 64 grid: launches and host work count
        case("chern_2band_64x64", "wilson", "qwz", 1, 0, 0.0, 1, 64, 64, "fp64", True),
        # the quadrupole insulator's nested loop on 100 x 100 points, the size the paper plots
        case("bbh_nested_100x100", "nested", "bbh", 1, 0, 0.0, 1, 100, 100, "fp64", True),
        # the nested loop against kz of a 3D higher-order insulator: 21 planes in one batch (largest k-point count)
        case("choti_nested_21_planes", "nested", "choti", 1, 0, 0.0, 21, 100, 100, "mixed"),
        # a small supercell on a small grid, as in a first look at a disordered model
        case("bhz4_wilson_12x10", "wilson", "bhz", 4, 0, 1.0, 1, 12, 10, "fp64", True),
        # a 96-orbital Wannier-like request of the served stream, at the precision it is served with
        case("w96_wilson_32x32_refined", "wilson", "wannier", 96, 0, 0.0, 1, 32, 32, "refined"),
        # the smallest supercell request of the served stream
        case("bhz8_wilson_32x32_mixed", "wilson", "bhz", 8, 0, 1.0, 1, 32, 32, "mixed"),
        # vacancies make the orders ragged (332 orbitals, 166 bands), on an odd grid
        case("qwz13_flux_vacancies_17x15", "flux", "qwz", 13, 3, 0.5, 2, 17, 15, "fp64"),
        # disorder study: spin-resolved loop of four 10 x 10 supercells on 24 x 24 points, in double precision
        case("bhz10_spin_24x24_fp64", "spin", "bhz", 10, 0, 1.0, 4, 24, 24, "fp64"),
        # the benchmark's chunk of the same study: eight systems on the mixed path
        case("bhz10_spin_24x24_mixed", "spin", "bhz", 10, 0, 1.0, 8, 24, 24, "mixed"),
        # spin-resolved flux map of one such supercell at refined precision
        case("bhz9_spin_flux_20x20_refined", "spin_flux", "bhz", 9, 2, 0.8, 1, 20, 20, "refined"),
        # an order-1024 supercell in double precision on a coarse grid
        case("bhz16_wilson_16x16_fp64", "wilson", "bhz", 16, 0, 1.0, 1, 16, 16, "fp64"),
        # the largest order of the served stream (2304), on a coarse grid
        case("bhz24_wilson_12x16_mixed", "wilson", "bhz", 24, 0, 1.0, 1, 12, 16, "mixed"),
    ]


def orbitals(c):
    return c["L"] if c["model"] == "wannier" else ORBITALS[c["model"]] * (c["L"] ** 2 - c["vacancies"])


def draw(rng):
    def spread(lo, hi):
        return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo - 0.49), math.log(hi + 0.49)))))))

    while True:
        call = rng.choice(["wilson", "wilson", "wilson", "spin", "spin", "flux", "spin_flux", "nested"])
        vac, dis, systems, L = 0, 0.0, 1, 1
        precision = rng.choice(["fp64", "fp64", "mixed", "refined"])
        n_perp, n_par = spread(8, 40), spread(6, 40)
        if call == "nested":
            model = rng.choice(["bbh", "choti"])
            systems = spread(2, 21) if model == "choti" else 1
            n_perp, n_par = spread(16, 100), spread(16, 100)
        else:
            model = {"wilson": rng.choice(["bhz", "bhz", "qwz", "wannier"]), "flux": "qwz"}.get(call, "bhz")
            systems = spread(1, 8)
        if model == "wannier":
            L, systems = spread(12, 128), min(systems, 3)
            precision = rng.choice(["fp64", "refined"])  # the mixed path misses its accuracy gate on this model
        elif model in ("bhz", "qwz"):
            L = spread(2, 24 if model == "bhz" else 30)
            dis = round(rng.uniform(0.3, 1.5), 3)
            vac = rng.choice([0, 0, int(round(0.02 * L * L))])
        c = case("", call, model, L, vac, dis, systems, n_perp, n_par, precision, rng.random() < 0.3)
        mats = systems * n_perp * n_par
        cost = mats * (orbitals(c) + 60) ** 3 * {"fp64": 2.0, "mixed": 1.0, "refined": 2.2}[precision]
        if cost < 0.6 * 256 * 2304.0 ** 3 and mats * orbitals(c) ** 2 * 16 < 12e9:
            return c


# ---------------------------------------------------------------- inputs


@dataclass
class Hoppings:
    """A hopping list as the engine takes it: amplitude t from orbital j in the
    cell at R to orbital i in the home cell, both Hermitian partners listed."""
    N: int
    dim: int
    i: np.ndarray
    j: np.ndarray
    R: np.ndarray
    t: np.ndarray


def unit_cell(model, rng):
    """{R: block} with one of each pair R, -R, and on-site random terms."""
    if model == "qwz":
        return {(0, 0): rng.uniform(0.8, 1.2) * S3, (1, 0): 0.5 * S3 + S1 / 2j, (0, 1): 0.5 * S3 + S2 / 2j}
    a = rng.standard_normal((4, 4)) + 1j * rng.standard_normal((4, 4))
    tilt = 0.02 * (a + a.conj().T)
    s3, s2 = np.kron(S3, S0), np.kron(S2, S0)
    if model == "bhz":
        return {(0, 0): rng.uniform(1.4, 1.6) * s3, (1, 0): 0.5 * s3 + np.kron(S1, S1) / 2j,
                (0, 1): 0.5 * s3 + np.kron(S1, S2) / 2j}
    if model == "bbh":
        g1, g2, g3, g4 = -np.kron(S2, S1), -np.kron(S2, S2), -np.kron(S2, S3), np.kron(S1, S0)
        return {(0, 0): rng.uniform(0.4, 0.6) * (g4 + g2) + tilt, (1, 0): 0.5 * g4 + g3 / 2j, (0, 1): 0.5 * g2 + g1 / 2j}
    return {(0, 0, 0): -1.5 * s3 + tilt, (1, 0, 0): 0.5 * s3 + np.kron(S1, S1) / 2j + 0.5 * s2,
            (0, 1, 0): 0.5 * s3 + np.kron(S1, S2) / 2j - 0.5 * s2, (0, 0, 1): 0.5 * s3 + np.kron(S1, S3) / 2j}


def both_partners(blocks):
    out = {}
    for R, T in blocks.items():
        out[R] = T
        if any(R):
            out[tuple(-r for r in R)] = T.conj().T
    return out


def from_blocks(blocks):
    cols = [[], [], [], []]
    for R, T in both_partners(blocks).items():
        a, b = np.nonzero(T)
        for col, v in zip(cols, (a, b, np.tile(np.array(R), (a.size, 1)), T[a, b])):
            col.append(v)
    i, j, R, t = (np.concatenate(v) for v in cols)
    return Hoppings(T.shape[0], R.shape[1], i.astype(np.int32), j.astype(np.int32), R.astype(np.int32), t)


def supercell(blocks, L, vacancies, disorder, rng):
    """L x L cells folded into one, some sites removed, a random scalar on every site."""
    n = next(iter(blocks.values())).shape[0]
    kept = np.sort(rng.permutation(L * L)[vacancies:])
    place = np.full(L * L, -1)
    place[kept] = np.arange(kept.size)
    x, y = kept // L, kept % L
    ii, jj, RR, tt = [], [], [], []
    for (rx, ry), T in both_partners(blocks).items():
        sx, sy = x + rx, y + ry
        to = place[(sx % L) * L + sy % L]
        ok = to >= 0
        here, to, cell = place[kept][ok], to[ok], np.stack([sx // L, sy // L], 1)[ok]
        for a, b in zip(*np.nonzero(T)):
            ii.append(n * here + a)
            jj.append(n * to + b)
            RR.append(cell)
            tt.append(np.full(here.size, T[a, b]))
    every = np.arange(n * kept.size)
    ii.append(every)
    jj.append(every)
    RR.append(np.zeros((every.size, 2), dtype=np.int64))
    tt.append(np.repeat(rng.uniform(-disorder / 2, disorder / 2, kept.size), n).astype(np.complex128))
    return Hoppings(n * kept.size, 2, np.concatenate(ii).astype(np.int32), np.concatenate(jj).astype(np.int32),
                    np.concatenate(RR).astype(np.int32), np.concatenate(tt))


def wannier_like(n, rng):
    """Random hoppings between n orbitals, decaying over the lattice vectors up to length 3."""
    blocks = {}
    for a in range(-3, 4):
        for b in range(-3, 4):
            if a * a + b * b <= 9 and (a, b) >= (0, 0):
                T = math.exp(-math.hypot(a, b) / 1.5) / math.sqrt(2) * (rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n)))
                blocks[(a, b)] = T if a or b else 0.5 * (T + T.conj().T)
    return from_blocks(blocks)


def inputs(c, seed):
    """Hopping lists and the k-grid, [n_perp, n_par, 3] (a stack of them for the planes of a 3D model)."""
    rng = np.random.default_rng([seed, 7])
    if c["model"] == "wannier":
        hops = [wannier_like(c["L"], rng) for _ in range(c["systems"])]
    elif c["model"] in ("bbh", "choti"):
        hops = [from_blocks(unit_cell(c["model"], rng))]
    else:
        cell = unit_cell(c["model"], rng)
        hops = [supercell(cell, c["L"], c["vacancies"], c["disorder"], rng) for _ in range(c["systems"])]
    off = rng.uniform(0.0, 1.0, 3)
    k = np.zeros((c["n_perp"], c["n_par"], 3))
    k[..., 0] = off[0] + np.arange(c["n_par"]) / c["n_par"]
    k[..., 1] = off[1] + (np.arange(c["n_perp"]) / c["n_perp"])[:, None]
    if c["model"] == "choti":
        k = np.repeat(k[None], c["systems"], 0)
        k[..., 2] = (off[2] + np.arange(c["systems"]) / c["systems"])[:, None, None]
    return hops, k


_context = None


def context():
    """One context for the program, as its users keep it."""
    global _context
    if _context is None:
        _context = _lib.Context(0)
    return _context


def prepare(c, seed):
    hops, k = inputs(c, seed)
    ctx = context()
    st = {"case": c, "ctx": ctx, "hops": hops, "k": k, "m": orbitals(c) // 2}
    st["plan"] = None if c["whole"] or c["model"] == "choti" else ctx.hk_plan(hops)
    st["spin"] = np.stack([np.tile(SPIN_BHZ, h.N // 4) for h in hops]) if c["call"].startswith("spin") else None
    return st


# ---------------------------------------------------------------- one pass

FIELDS = {
    "wilson": ("theta", "phi", "winding", "status"),
    "nested": ("theta", "s", "p", "p_mean", "status"),
    "spin": ("mu", "theta_dn", "theta_up", "m_dn", "C_dn", "C_up", "C_s", "status"),
    "flux": ("flux", "chern", "total", "status"),
    "spin_flux": ("mu", "m_dn", "flux_dn", "flux_up", "C_dn", "C_up", "C_s", "total_dn", "total_up", "status"),
}


def run(st):
    c, ctx, hops, k, m = st["case"], st["ctx"], st["hops"], st["k"], st["m"]
    call, precision = c["call"], PRECISION[c["precision"]]
    if c["model"] == "choti":
        out = pipeline.wnwl_planes(ctx, hops[0], k, 0, m, precision=precision)
    elif c["whole"] and call == "wilson":
        out = pipeline.wsurf(ctx, hops, k, 0, m, precision=precision)
    elif c["whole"] and call == "nested":
        out = pipeline.wnwl(ctx, hops, k, 0, m, precision=precision)
    elif c["whole"] and call == "spin":
        out = pipeline.wspinsurf(ctx, hops, st["spin"], k, 0, m, precision=precision)
    elif c["whole"] and call == "flux":
        out = pipeline.wflux(ctx, hops, k, 0, m, precision=precision)
    elif c["whole"]:
        out = pipeline.wspinflux(ctx, hops, st["spin"], k, 0, m, precision=precision)
    else:
        g = pipeline.eig_grid(ctx, st["plan"], 0, c["systems"], k, 0, m, precision,
                              chunk=c["systems"] * c["n_perp"] * c["n_par"])
        if call == "wilson":
            out = pipeline.wilson(ctx, g)
        elif call == "nested":
            out = pipeline.nested(ctx, g)
        elif call == "spin":
            out = pipeline.spin(ctx, g, st["spin"], precision=precision)
        elif call == "flux":
            out = pipeline.flux(ctx, g)
        else:
            out = pipeline.spin_flux(ctx, g, st["spin"], precision)
        out["eig"] = g
    return dict({f: out[f] for f in FIELDS[call]}, evals=out["eig"].evals, eig_status=out["eig"].status)


def work(c):
    """Bytes: the hopping lists and k-points in, the results out. Operations
    (8 a complex multiply-add): the reduction to tridiagonal form and the
    vectors of the occupied bands, then per link its overlap, polar factor
    (one inversion's worth) and product, or its determinant."""
    N, planes = orbitals(c), c["systems"]
    m, mats = N // 2, c["systems"] * c["n_perp"] * c["n_par"]
    entries = 29 * N * N if c["model"] == "wannier" else 16 * N
    eig = 16 / 3 * N ** 3 + 8 * N * N * m
    loop = {"wilson": 8 * N * m * m + 24 * m ** 3, "flux": 2 * (8 * N * m * m + 8 / 3 * m ** 3)}
    loop["nested"] = loop["wilson"] + 8 * N * m
    sectors = 8 * N * m * m + 16 / 3 * m ** 3 + 8 * m ** 3 + 8 * N * m * m
    loop["spin"] = sectors + 2 * (8 * N * (m / 2) ** 2 + 24 * (m / 2) ** 3)
    loop["spin_flux"] = sectors + 4 * (8 * N * (m / 2) ** 2 + 8 / 3 * (m / 2) ** 3)
    lines = c["systems"] * c["n_perp"]
    out = mats * (m + 2) * 8 + {"wilson": lines * m * 8, "nested": c["systems"] * c["n_par"] * (m + 1) * 8,
                                "spin": mats * m * 8 + 2 * lines * m * 8, "flux": mats * 8,
                                "spin_flux": mats * m * 8 + 2 * mats * 8}[c["call"]]
    return {"bytes": float(planes * entries * 32 + mats * 24 + out), "flops": float(mats * (eig + loop[c["call"]]))}


# ---------------------------------------------------------------- the same in plain 64-bit torch


def solve(hops, k, m):
    """Eigenvalues [lo - 1, hi] as the engine lays them out, and the occupied vectors, [n, N, m]."""
    ev, U = [], []
    kt = torch.from_numpy(k.reshape(-1, 3))
    for h in hops:
        cells, at = np.unique(h.R, axis=0, return_inverse=True)
        T = torch.zeros(len(cells) * h.N * h.N, dtype=torch.complex128)
        T.index_add_(0, torch.from_numpy((at.reshape(-1) * h.N + h.i) * h.N + h.j), torch.from_numpy(h.t))
        ph = torch.exp(2j * math.pi * (kt[:, :h.dim] @ torch.from_numpy(cells.astype(np.float64)).T.contiguous()))
        H = (ph @ T.view(len(cells), -1)).view(-1, h.N, h.N)
        H = 0.5 * (H + H.mH)
        w, V = map(torch.from_numpy, np.linalg.eigh(H.numpy()))
        nan = torch.full((len(w), 1), math.nan, dtype=torch.float64)
        ev.append(torch.cat([nan, w[:, :m + 1], nan][: 2 if m < h.N else 3], 1))
        U.append(V[:, :, :m].contiguous())
    return torch.cat(ev), torch.cat(U)


def polar(F):
    X, _, Yh = np.linalg.svd(F.numpy())
    return torch.from_numpy(X @ Yh)


def links(U, along):
    """U(next)^H U of a grid [lines, points, N, m], the points of `along` closed."""
    return torch.roll(U, -1, along).mH.contiguous() @ U


def loop_matrices(F):
    W = F[:, 0]
    for j in range(1, F.shape[1]):
        W = F[:, j] @ W
    return W


def phases(W):
    return torch.from_numpy(np.sort(np.angle(np.linalg.eigvals(W.numpy())), -1))


def wrap(x):
    return x - 2 * math.pi * torch.round(x / (2 * math.pi))


def nested_exact(U, n_perp, n_par):
    """One system: nested phases per base point, their sum as a polarization, its mean."""
    F = polar(links(U, 1))
    lam, nu = np.linalg.eig(loop_matrices(F).numpy())
    x = np.angle(lam) / (2 * math.pi)
    inside = (x > 0) & (x < 0.5)
    s = int(inside[0].sum())
    q = np.linalg.qr(np.stack([v[:, g] for v, g in zip(nu, inside)]))[0]
    q, carried = torch.from_numpy(q), []
    for j in range(n_par):
        carried.append(U[:, j] @ q)
        q = F[:, j] @ q
    th = phases(loop_matrices(polar(links(torch.stack(carried), 1))))
    out = torch.full((n_par, U.shape[-1]), math.nan, dtype=torch.float64)
    out[:, :s] = th
    p = th.sum(-1) / (2 * math.pi)
    p = p - torch.round(p)
    step = p[1:] - p[:-1]
    whole = torch.cat([p[:1], step - torch.round(step)]).cumsum(0)
    return out, p, whole.mean() % 1.0


def flux_exact(U):
    """One system's grid: flux through every plaquette and its sum over 2 pi."""
    a, b = (torch.angle(torch.linalg.slogdet(links(U, d))[0]) for d in (1, 0))
    f = wrap(torch.roll(a, -1, 0) - a + b - torch.roll(b, -1, 1))
    return f, f.sum() / (2 * math.pi)


def exact(c, seed):
    N = orbitals(c)
    m, mats = N // 2, c["systems"] * c["n_perp"] * c["n_par"]
    if mats * (N + 12) ** 3 > 2.5e10:  # over about 20 seconds
        return None
    hops, k = inputs(c, seed)
    grids = c["systems"], c["n_perp"], c["n_par"]
    ev, U = solve(hops, k, m)
    U = U.view(*grids, N, m)
    out = dict.fromkeys(FIELDS[c["call"]] + ("evals", "eig_status"), None)
    out["evals"] = ev
    if c["call"] == "wilson":
        th = torch.stack([phases(loop_matrices(polar(links(u, 1)))) for u in U])
        out.update(theta=th, phi=th.sum(-1) % (2 * math.pi))
    elif c["call"] == "nested":
        got = [nested_exact(u, c["n_perp"], c["n_par"]) for u in U]
        out.update(zip(("theta", "p", "p_mean"), (torch.stack(v) for v in zip(*got))))
    elif c["call"] == "flux":
        out.update(zip(("flux", "total"), (torch.stack(v) for v in zip(*(flux_exact(u) for u in U)))))
    else:
        S = torch.from_numpy(np.tile(SPIN_BHZ, N // 4))
        mu, Q = map(torch.from_numpy, np.linalg.eigh((U.mH @ (S[:, None] * U)).numpy()))
        V = U @ Q
        dn = int((mu[0, 0, 0] < 0).sum())
        out["mu"] = mu if c["call"] == "spin" else mu.reshape(*grids, m)
        for key, part in (("dn", V[..., :dn].contiguous()), ("up", V[..., dn:].contiguous())):
            if c["call"] == "spin":
                th = torch.full((*grids[:2], m), math.nan, dtype=torch.float64)
                for s, u in enumerate(part):
                    th[s, :, :u.shape[-1]] = phases(loop_matrices(polar(links(u, 1))))
                out["theta_" + key] = th
            else:
                got = [torch.stack(v) for v in zip(*(flux_exact(u) for u in part))]
                out["flux_" + key], out["total_" + key] = got
    return out
