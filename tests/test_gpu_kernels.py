"""GPU parity of the kernels chosen by shape: each at the sizes where its split, tile or
remainder can go wrong, against the FP64 oracle (relative L2 <= 1e-5, the bar of the path)."""
import numpy as np
import pytest

import synth
from oracle import oracle as O
from tests.helpers import assert_parity, gpu_intensity

pytestmark = pytest.mark.gpu


def say(msg):
    print(f"[gpu case] {msg}", flush=True)


def sampled_parity(m, order=None, most=4000):
    """The model's box on the GPU against the oracle at (a sample of) its points."""
    I = gpu_intensity(m)
    G = O.grid_points(m.g0, m.count)
    if len(G) > most:
        G = G[np.random.default_rng(1).choice(len(G), most, replace=False)]
    got, ref = I[tuple((G - np.asarray(m.g0)).T)], O.intensity(m, G, order)
    if not np.any(ref):          # one configuration at unit-cell Bragg points only: exactly 0
        assert not np.any(got)
    else:
        assert_parity(got, ref)


# ------------------------------------------------------------------ register transforms n = A B
@pytest.mark.parametrize("n", [(14, 15, 9), (10, 6, 12), (11, 13, 16), (2, 1, 20), (1, 18, 2), (3, 5, 64), (40, 3, 2),
                               (2, 121, 6), (169, 2, 4), (5, 9, 143), (6, 96, 33), (2, 225, 5), (3, 2, 224), (27, 25, 21),
                               (17, 12, 10), (12, 34, 10), (10, 12, 19)])
@pytest.mark.parametrize("kind", [synth.NUCLEAR, synth.MAGNETIC])
def test_edges_of_two_factors(n, kind):
    """Every radix up to 16 in both passes, odd and even row counts, several planes per block,
    and edges with a prime factor above 16 beside them (those planes or columns take the
    Stockham passes)."""
    order = 2 if kind == synth.NUCLEAR else 0
    m = synth.random_model(900 + sum(n), n=n, S=2, M=2, order=order, kind=kind, sigma=0.03,
                           cell=None if kind == synth.NUCLEAR else [6.0, 7.0, 8.0, 90.0, 90.0, 90.0])
    m.g0 = tuple(-min(v + 1, 12) for v in n)
    m.count = tuple(min(2 * v + 3, 25) for v in n)
    say(f"two-factor edges n={n} kind={kind}")
    sampled_parity(m, order if kind == synth.NUCLEAR else None)


def test_plane_rows_route_of_two_factor_edges():
    """A plane past the LDS budget: rows along axis 3 per block, then axis 2 in place."""
    m = synth.random_model(961, n=(2, 196, 208), S=1, M=1, order=1, sigma=0.03)
    m.g0, m.count = (-2, -9, -9), (5, 19, 19)
    say(f"row route n={m.n}")
    sampled_parity(m, 1, 1500)


# ------------------------------------------------------------------ recombination, sites form
def sites_model(seed, n, S, M, order, r3=None, ff=False, occ=True):
    m = synth.random_model(seed, n=n, S=S, M=M, order=order, with_occ=occ or order == 0, with_disp=order > 0, sigma=0.03)
    if r3 is not None:
        m.frac[:, 2] = np.asarray(r3)[np.arange(S) % len(r3)]
    if ff:
        m.ff = np.tile(synth.MAG_FF, (S, 1))
        m.ff[:, 6] = 0.2 + 0.1 * (np.arange(S) % 2)
    return m


@pytest.mark.parametrize("S,M,order,r3", [(1, 3, 2, None), (5, 1, 0, None), (33, 2, 0, None), (7, 40, 0, (0.1, 0.6, 0.1)),
                                          (3, 9, 4, (0.0, 0.5)), (4, 2, 8, (0.25, 0.3)), (64, 1, 1, None), (2, 5, 11, None)])
@pytest.mark.parametrize("box", ["symmetric", "plane1", "plane2", "plane3", "thin3", "offset"])
def test_sites_form(S, M, order, r3, box):
    """Configurations side by side, site chunks, shared and separate r3 classes, parity sets, and
    boxes with one plane per axis, fewer G3 than the supercell has k3, or none symmetric."""
    n = (4, 3, 5) if order > 8 else (5, 4, 18)
    m = sites_model(2000 + S + M + order, n, S, M, order, r3)
    lim = {"symmetric": [(-n[a] - 1, 2 * n[a] + 3) for a in range(3)], "offset": [(-3, n[0] + 2), (1, n[1] + 3), (-n[2] - 4, 2 * n[2] + 1)]}
    full = [(-n[a] - 2, 2 * n[a] + 4) for a in range(3)]
    for a in range(3):
        lim[f"plane{a + 1}"] = full[:a] + [(n[a] + 1, 1)] + full[a + 1:]
    lim["thin3"] = full[:2] + [(n[2] - 2, 4)]
    m.g0, m.count = tuple(v[0] for v in lim[box]), tuple(v[1] for v in lim[box])
    say(f"sites form S={S} M={M} order={order} box={m.g0}+{m.count}")
    sampled_parity(m, order if order else None, 1500)


@pytest.mark.parametrize("n3,M", [(15, 1), (16, 7), (47, 2), (64, 1)])
def test_sites_form_scattering_factors(n3, M):
    """Slices of k3 (n3 >= 16) with |Q|-dependent factors in the class form."""
    m = sites_model(2200 + n3, (3, 4, n3), 4, M, 3, (0.2, 0.7), ff=True)
    m.cell = np.array([5.0, 6.0, 7.0, 90.0, 97.0, 90.0])
    m.g0, m.count = (-4, -5, -n3 - 3), (9, 11, 2 * n3 + 7)
    say(f"sites form with factors n={m.n} M={M}")
    sampled_parity(m, 3, 1500)


# ------------------------------------------------------------------ points: rows of the windows only
@pytest.mark.parametrize("shape", ["hhl", "line", "off"])
@pytest.mark.parametrize("kind,S,M,order,basis", [("occ", 6, 20, 0, None), ("disp", 4, 1, 3, "fcc"), ("disp", 3, 2, 2, None),
                                                  ("mag", 4, 1, 0, "fcc"), ("mag", 2, 2, 0, None), ("mag", 2, 1, 2, None)])
def test_points_cut_work_lists(shape, kind, S, M, order, basis):
    """Planes, lines and one-sided sets of points, whose windows reach few rows of their box: every
    form's work list cut down to them (mirrored and paired planes among them)."""
    import torch
    from tests.helpers import to_dsx
    magnetic = kind == "mag"
    m = synth.random_model(2300 + S + M + order, n=(6, 5, 8), S=S, M=M, order=order, kind=synth.MAGNETIC if magnetic else synth.NUCLEAR,
                           with_occ=kind == "occ", with_disp=order > 0, mag_order=order if magnetic else 0, sigma=0.03,
                           cell=[6.0, 6.0, 6.0, 90.0, 90.0, 90.0] if magnetic else None)
    if basis == "fcc":
        m.frac = synth.FCC_BASIS[:S].copy()
    t = np.linspace(-2.3, 2.3, 9)
    h, l = (v.ravel() for v in np.meshgrid(t, t, indexing="ij"))
    Q = {"hhl": np.stack([6 * h, 5 * h, 8 * l], -1), "line": np.stack([6 * t, 0 * t + 1.5, 8 * t], -1),
         "off": np.stack([6 * h + 31.25, -5 * h - 20.5, 8 * l], -1)}[shape]
    say(f"points {shape} {kind} S={S} M={M} order={order}")
    d = to_dsx(m)
    out = torch.full((len(Q),), float("nan"), dtype=torch.float32, device="cuda")
    d.filter_points(2, Q, out)
    got = out.cpu().numpy()
    d.close()
    assert_parity(got, O.filtered_points(m, 2, Q, order if order and not magnetic else None))


@pytest.mark.parametrize("shape", ["hhl", "line", "off"])
@pytest.mark.parametrize("kind,S,M,order,basis", [("occ", 6, 20, 0, None), ("disp", 4, 4, 3, "fcc"), ("disp", 3, 6, 2, None),
                                                  ("mag", 4, 6, 0, "fcc"), ("mag", 2, 10, 0, None), ("mag", 2, 10, 2, None)])
def test_points_cut_work_lists_of_wide_boxes(shape, kind, S, M, order, basis):
    """The same over boxes of 17 000 rows, which hold enough terms that the lists are worth cutting,
    against the call whose points reach every row of the box."""
    import torch
    from tests.helpers import to_dsx
    magnetic = kind == "mag"
    m = synth.random_model(2350 + S + M + order, n=(6, 5, 8), S=S, M=M, order=order, kind=synth.MAGNETIC if magnetic else synth.NUCLEAR,
                           with_occ=kind == "occ", with_disp=order > 0, mag_order=order if magnetic else 0, sigma=0.03,
                           cell=[6.0, 6.0, 6.0, 90.0, 90.0, 90.0] if magnetic else None)
    if basis == "fcc":
        m.frac = synth.FCC_BASIS[:S].copy()
    t = np.linspace(-12.1, 12.1, 9)
    h, l = (v.ravel() for v in np.meshgrid(t, t / 3, indexing="ij"))
    Q = {"hhl": np.stack([6 * h, 5 * h, 8 * l], -1), "line": np.stack([6 * t, 5 * t + 0.5, 8 * t / 3], -1),
         "off": np.stack([6 * h + 131.25, -5 * h - 20.5, 8 * l], -1)}[shape]
    say(f"points over a wide box {shape} {kind} S={S} M={M} order={order}")
    d = to_dsx(m)
    step = [np.arange(*np.floor(Q[:, a])[[0, -1]][np.argsort(Q[[0, -1], a])], 3) + 0.5 for a in (0, 1)]
    cover = np.stack([v.ravel() for v in np.meshgrid(*step, Q[:1, 2], indexing="ij")], -1)
    got = []
    for q in (Q, np.concatenate([Q, cover])):
        out = torch.full((len(q),), float("nan"), dtype=torch.float32, device="cuda")
        d.filter_points(2, q, out)
        got.append(out.cpu().numpy())
    d.close()
    assert np.isfinite(got[1]).all()
    assert_parity(got[0], got[1][:len(Q)])


# ------------------------------------------------------------------ Bragg points of ensembles
@pytest.mark.parametrize("S,M,order", [(20, 64, 0), (3, 65, 0), (17, 130, 0), (2, 40, 2)])
def test_bragg_points_of_ensembles(S, M, order):
    """Lanes over the configurations: whole and ragged multiples of the wave, 1 to 64 sites."""
    m = synth.random_model(2400 + S + M, n=(2, 3, 2), S=S, M=M, order=order, with_occ=True, with_disp=order > 0, sigma=0.03)
    m.g0, m.count = (-4, -6, -4), (9, 13, 9)
    say(f"Bragg ensemble S={S} M={M} order={order}")
    I = gpu_intensity(m).reshape(m.count)[::2, ::3, ::2]
    G = O.grid_points(m.g0, m.count).reshape(m.count + (3,))[::2, ::3, ::2].reshape(-1, 3)
    assert_parity(I.reshape(-1), O.intensity(m, G, order if order else None))


@pytest.mark.parametrize("S,M", [(1, 16), (2, 17), (1, 70), (5, 16)])
def test_many_bragg_points_of_ensembles(S, M):
    """Boxes of 1331 Bragg points: lanes over the points for few terms, else over the configurations."""
    m = synth.random_model(2450 + S + M, n=(2, 3, 2), S=S, M=M, order=0, with_occ=True, with_disp=False)
    m.g0, m.count = (-10, -15, -10), (21, 31, 21)
    say(f"many Bragg points of an ensemble S={S} M={M}")
    I = gpu_intensity(m).reshape(m.count)[::2, ::3, ::2]
    G = O.grid_points(m.g0, m.count).reshape(m.count + (3,))[::2, ::3, ::2].reshape(-1, 3)
    assert_parity(I.reshape(-1), O.intensity(m, G, None))


# ------------------------------------------------------------------ one site: tiled rows
@pytest.mark.parametrize("n,M", [((3, 4, 5), 1), ((12, 5, 7), 3), ((2, 3, 31), 70), ((9, 8, 64), 2), ((1, 2, 200), 1)])
@pytest.mark.parametrize("box", ["symmetric", "offset", "short"])
@pytest.mark.parametrize("lm", [0, 2])
def test_one_site_tiles(n, M, box, lm):
    """Dense rows of any length mod 4 and padded rows (under the filter), half-stored boxes, rows
    shorter than the supercell, several configurations over the threads."""
    from tests.helpers import gpu_filtered
    m = synth.random_model(2500 + sum(n) + M, n=n, S=1, M=M, order=0, with_disp=False)
    r = [min(v + 2, 9) for v in n]
    m.g0, m.count = {"symmetric": ([-v for v in r], [2 * v + 1 for v in r]), "offset": ([-v for v in r], [2 * v + 2 for v in r]),
                     "short": ([-r[0], -r[1], n[2] - 2], [2 * r[0] + 1, 2 * r[1] + 1, 3])}[box]
    m.g0, m.count = tuple(m.g0), tuple(m.count)
    say(f"one site n={n} M={M} box={m.g0}+{m.count} lm={lm}")
    if lm:
        assert_parity(gpu_filtered(m, lm), O.filtered_intensity(m, lm, 1))
    else:
        sampled_parity(m)


# ------------------------------------------------------------------ filter: oversampled and wide windows
@pytest.mark.parametrize("lm,mp,s", [(2, 2, 2), (2, 2, 3), (3, 2, 2), (4, 2, 5), (2, 3, 16), (5, 2, 1), (5, 2, 2), (4, 3, 1),
                                     (7, 2, 1), (4, 4, 1), (8, 2, 3), (3, 6, 2), (6, 3, 1)])
@pytest.mark.parametrize("count", [(3, 9, 33), (14, 5, 2)])
def test_oversampled_and_wide_filters(lm, mp, s, count):
    """Every window width of the streaming kernel (and one past it), phases that do and do not
    divide the tile, ragged tiles and segments, a half-stored and an unsymmetric box."""
    from tests.helpers import gpu_filtered
    m = synth.random_model(2600 + lm + mp + s, n=(3, 4, 5), S=1, M=2, order=0, with_disp=False)
    m.count = count
    m.g0 = tuple(-(c - 1) // 2 if c % 2 else -1 for c in count)
    say(f"filter m={lm} m'={mp} s={s} box={m.g0}+{m.count}")
    assert_parity(gpu_filtered(m, lm, s, mp), O.filtered_intensity(m, lm, s, mprime=mp))


# ------------------------------------------------------------------ magnetic, Debye-Waller rows form
@pytest.mark.parametrize("S,M,order,n", [(1, 1, 1, (3, 4, 5)), (3, 4, 2, (4, 3, 6)), (5, 9, 3, (3, 3, 4)), (2, 2, 16, (2, 3, 3)),
                                         (20, 3, 2, (2, 2, 9)), (64, 1, 3, (1, 2, 40)), (16, 5, 4, (2, 1, 64))])
@pytest.mark.parametrize("box", ["symmetric", "offset", "long"])
def test_debye_waller_rows(S, M, order, n, box):
    """One, two and four configurations a pass, ragged last passes, uniform and separate form
    factors, few rows a block, and G3 ranges past the threads of a block (the other form)."""
    m = synth.random_model(2700 + S + M + order, n=n, S=S, M=M, kind=synth.MAGNETIC, mag_order=order, sigma=0.03,
                           cell=[5.0, 6.0, 7.0, 90.0, 97.0, 90.0])
    if S % 2:
        m.ff[::2, 6] = 0.3
    r = [v + 1 for v in n]
    m.g0, m.count = {"symmetric": ([-v for v in r], [2 * v + 1 for v in r]), "offset": ([1, -r[1], -2], [r[0], 2 * r[1], n[2] + 3]),
                     "long": ([0, 0, -2], [2, 2, 515])}[box]
    if box == "long" and (n[2] > 9 or n[2] * -(-515 // n[2] // 17) > 512):
        m.count[2] = 4 * n[2]
    m.g0, m.count = tuple(m.g0), tuple(m.count)
    say(f"Debye-Waller rows S={S} M={M} order={order} n={n} box={m.g0}+{m.count}")
    sampled_parity(m, None, 1200)


# ------------------------------------------------------------------ magnetic rows, several configurations
@pytest.mark.parametrize("S,M,r", [(4, 2, 0.5), (4, 3, 0.5), (8, 4, 0.25), (3, 5, 1 / 3), (5, 9, None), (64, 2, None), (2, 6, 1.0)])
@pytest.mark.parametrize("n", [(4, 3, 6), (3, 2, 64)])
@pytest.mark.parametrize("box", ["symmetric", "offset", "wide"])
def test_magnetic_rows_configurations(S, M, r, n, box):
    """One, two and four configurations a pass, one and several passes, planes grouped (sites on a
    grid) and not, residue sums and separate classes."""
    m = synth.random_model(2800 + S + M, n=n, S=S, M=M, kind=synth.MAGNETIC, cell=[6.0, 7.0, 8.0, 90.0, 90.0, 90.0])
    if r is not None:
        m.frac = np.round(m.frac / r) * r
    m.g0, m.count = {"symmetric": ([-9, -7, -n[2] - 2], [19, 15, 2 * n[2] + 5]), "offset": ([2, -5, 1], [14, 9, n[2]]),
                     "wide": ([-1, -1, -150], [3, 3, 300 if S == 64 else 500])}[box]
    m.g0, m.count = tuple(m.g0), tuple(m.count)
    say(f"magnetic rows S={S} M={M} grid={r} n={n} box={m.g0}+{m.count}")
    sampled_parity(m, None, 1500)


@pytest.mark.parametrize("S,M,n", [(10, 3, (2, 3, 62)), (6, 3, (3, 4, 12)), (3, 6, (4, 3, 20)), (15, 2, (2, 3, 45)), (24, 1, (2, 2, 62))])
def test_magnetic_rows_staged_one_by_one(S, M, n):
    """Sites off every grid: one or two configurations a pass, the rows a block holds bounded by the
    LDS that three blocks of a compute unit share, down to one."""
    m = synth.random_model(2870 + S + M, n=n, S=S, M=M, kind=synth.MAGNETIC, cell=[6.0, 7.0, 8.0, 90.0, 90.0, 90.0])
    m.g0, m.count = (-n[0], -3 * n[1] - 1, -n[2] - 1), (2 * n[0] + 1, 6 * n[1] + 3, 2 * n[2] + 3)
    say(f"staged magnetic rows S={S} M={M} n={n}")
    sampled_parity(m, None, 1500)


@pytest.mark.parametrize("r,S,M", [(4, 16, 2), (4, 16, 3), (4, 16, 5), (2, 16, 3), (4, 8, 3), (2, 12, 2)])
@pytest.mark.parametrize("box", ["symmetric", "offset"])
def test_magnetic_rows_of_many_columns(r, S, M, box):
    """Passes of one configuration over 3240 columns and more, whose sums are in LDS, and passes of
    all configurations whose planes share a block; sites on quarters and halves."""
    m = synth.random_model(4000 + S + M + r, n=(10, 40, 40), S=S, M=M, order=0, kind=synth.MAGNETIC, with_disp=False,
                           cell=[6.0, 6.0, 6.0, 90.0, 90.0, 90.0])
    m.frac = np.random.default_rng(S + r).integers(0, r, m.frac.shape) / r
    m.g0, m.count = ((-80, -60, -120), (161, 121, 241)) if box == "symmetric" else ((-77, -50, -110), (79, 100, 230))
    say(f"magnetic rows of many columns r={r} S={S} M={M} box={m.g0}+{m.count}")
    sampled_parity(m, most=200)


# ------------------------------------------------------------------ lines of a prime length
@pytest.mark.parametrize("p", [17, 19, 23, 29, 31, 37, 41, 43, 47, 53, 59, 61, 67])
@pytest.mark.parametrize("axis", [0, 1, 2])
def test_prime_edges(p, axis):
    """Every prime past the small radices on every axis, alone and times 2 to 4 (67: the Stockham
    passes)."""
    f = 1 + p % 4 if p < 60 else 1
    n = [3, 2, 4]
    n[axis] = p * f
    m = synth.random_model(2900 + p + axis, n=tuple(n), S=2, M=2, order=1, sigma=0.03)
    m.g0 = tuple(-min(v + 1, 30) for v in n)
    m.count = tuple(min(2 * v + 3, 63) for v in n)
    say(f"prime edges n={m.n}")
    sampled_parity(m, 1, 1000)


# ------------------------------------------------------------------ boxes transformed whole
@pytest.mark.parametrize("n", [(1, 1, 1), (2, 1, 3), (16, 16, 16), (13, 9, 11), (5, 16, 1), (12, 12, 12), (7, 2, 15)])
@pytest.mark.parametrize("kind,order,M,occ", [(synth.NUCLEAR, 0, 3, True), (synth.NUCLEAR, 3, 1, False), (synth.NUCLEAR, 8, 2, True),
                                              (synth.MAGNETIC, 0, 2, False)])
def test_whole_boxes(n, kind, order, M, occ):
    """Edges up to 16: generation and the three axes in one block, with and without
    the constant monomial, one field and ragged chunks of fields."""
    m = synth.random_model(3000 + sum(n) + order, n=n, S=2, M=M, order=order, kind=kind, with_occ=occ, with_disp=order > 0, sigma=0.03,
                           cell=None if kind == synth.NUCLEAR else [6.0, 7.0, 8.0, 90.0, 90.0, 90.0])
    m.g0 = tuple(-(v // 2) - 2 for v in n)
    m.count = tuple(v + 5 for v in n)
    say(f"whole box n={n} kind={kind} order={order}")
    sampled_parity(m, order if order and kind == synth.NUCLEAR else None, 1200)


# ------------------------------------------------------------------ folded form on thin boxes
@pytest.mark.parametrize("order,M", [(2, 1), (3, 3), (6, 1), (7, 2), (8, 1)])
@pytest.mark.parametrize("n3,g3,c3", [(18, 5, 1), (18, -3, 5), (18, 15, 17), (6, 4, 4), (32, -16, 20)])
def test_folded_form_with_fewer_g3_than_k3(order, M, n3, g3, c3):
    """Boxes whose G3 leave some k3 without points (the active ones wrap around), sliced and not,
    with odd and even numbers of (q, r) pairs."""
    m = synth.random_model(3100 + order + n3, n=(3, 4, n3), S=4, M=M, order=order, with_occ=False, sigma=0.03)
    m.frac = synth.FCC_BASIS.copy()
    m.g0, m.count = (-4, -6, g3), (9, 12, c3)
    say(f"folded thin order={order} M={M} box={m.g0}+{m.count}")
    sampled_parity(m, order, 1500)


# ------------------------------------------------------------------ Bragg points of one configuration
@pytest.mark.parametrize("kind,order", [(synth.NUCLEAR, 0), (synth.NUCLEAR, 2), (synth.MAGNETIC, 0), (synth.MAGNETIC, 2)])
@pytest.mark.parametrize("bad", [None, np.nan, np.inf])
def test_bragg_points_of_one_configuration(kind, order, bad):
    """Exactly 0, and not a number where an input is not (but 0 at the origin of magnetic models)."""
    m = synth.random_model(3200 + order, n=(3, 4, 5), S=3, M=1, order=order, kind=kind, with_disp=order > 0, mag_order=order, sigma=0.03,
                           cell=None if kind == synth.NUCLEAR else [6.0, 7.0, 8.0, 90.0, 90.0, 90.0])
    m.g0, m.count = (-6, -8, -10), (13, 17, 21)
    if bad is not None:
        (m.spin if kind == synth.MAGNETIC else m.disp if order else m.occ)[0, 1, 0, 0, 0] = bad
    say(f"Bragg points of one configuration kind={kind} order={order} bad={bad}")
    I = gpu_intensity(m).reshape(m.count)[::3, ::4, ::5]
    if bad is None:
        assert not np.any(I)
    else:
        want = np.ones(I.shape, bool)
        if kind == synth.MAGNETIC:
            want[2, 2, 2] = False
        assert np.array_equal(np.isnan(I), want)


# ------------------------------------------------------------------ sites form: rows a group holds
@pytest.mark.parametrize("n,rows,c3,S,M,order,r3", [((2, 2, 64), 9, 131, 3, 1, 0, None), ((3, 15, 125), 5, 251, 4, 1, 3, (0.2, 0.7)),
                                                    ((2, 2, 32), 17, 65, 5, 1, 2, (0.0, 0.5)), ((2, 1, 50), 12, 53, 2, 3, 1, None),
                                                    ((2, 2, 16), 17, 640, 3, 1, 0, None), ((2, 1, 96), 6, 97, 2, 9, 0, None),
                                                    ((1, 2, 20), 32, 41, 3, 1, 5, None), ((2, 1, 24), 26, 49, 2, 2, 9, None)])
def test_sites_form_writes_every_row(n, rows, c3, S, M, order, r3):
    """Columns of so many rows that blocks of 320 items would pass the threads a plane of a
    two-plane block has: every voxel is written (the output starts as NaN)."""
    import torch
    from tests.helpers import to_dsx
    m = sites_model(3300 + S + M + order, n, S, M, order, r3)
    m.frac[:, 1] = 0.3 + 0.1 * np.arange(S)          # (no folding)
    m.g0 = (-2 * n[0], -((rows * n[1]) // 2), -(c3 // 2))
    m.count = (4 * n[0] + 1, rows * n[1], c3)
    say(f"sites form rows n={n} box={m.g0}+{m.count} S={S} M={M} order={order}")
    h = to_dsx(m)
    out = torch.full(m.count, float("nan"), dtype=torch.float32, device="cuda")
    h.compute_intensity(out)
    got = out.cpu().numpy()
    h.close()
    assert not np.any(np.isnan(got)), f"{int(np.isnan(got).sum())} voxels not written"
    G = O.grid_points(m.g0, m.count)
    pick = np.random.default_rng(1).choice(len(G), min(len(G), 4000), replace=False)
    assert_parity(got.reshape(-1)[pick], O.intensity(m, G[pick], order if order else None))


@pytest.mark.parametrize("kind,order", [(synth.NUCLEAR, 0), (synth.NUCLEAR, 5), (synth.MAGNETIC, 0), (synth.MAGNETIC, 2)])
@pytest.mark.parametrize("bad", ["b inf", "b nan", "b 1e160", "b 1e30", "ff inf", "ff grows", "disp 1e38"])
def test_bragg_points_of_one_configuration_with_extreme_weights(kind, order, bad):
    """Not a number where a weight is not finite or the squared structure factor overflows float64
    (there the subtraction of its two squares is inf - inf), exactly 0 everywhere else."""
    m = synth.random_model(3400 + order, n=(3, 4, 5), S=3, M=1, order=order, kind=kind, with_disp=order > 0, mag_order=order, sigma=0.03,
                           cell=[1.0, 1.1, 0.9, 90.0, 95.0, 90.0] if kind == synth.NUCLEAR else [6.0, 7.0, 8.0, 90.0, 90.0, 90.0])
    m.g0, m.count = (-6, -8, -10), (13, 17, 21)
    H = O.grid_points((-2, -2, -2), (5, 5, 5))
    want = np.zeros(len(H), bool)
    if bad.startswith("b "):
        m.b[1] = float(bad[2:])
        want[:] = bad != "b 1e30"
    elif bad == "disp 1e38":
        if order != 5:
            pytest.skip("needs a Taylor order whose powers pass 1e154 in the lattice sums")
        m.disp[0, 1, 0, 0, 0] = 1e38
        m.occ[0, 1, 0, 0, 0] = 1.0
        want[:] = np.any(H != 0, axis=1)     # (every power has the factor 0 at the origin)
    else:
        if m.ff is None:
            m.ff = np.tile(synth.MAG_FF, (3, 1))
        if bad == "ff inf":
            m.ff[1, 6] = np.inf
            want[:] = True
        else:
            # 0.4 exp(+B s^2): the first factor past 1e160 (none of them near) at the larger |H|
            cell = np.asarray(m.cell)
            scale = 1.0 if kind == synth.NUCLEAR else 50.0
            m.ff[1, 1] = -800.0 * scale
            a = np.diag(cell[:3])
            a[2] = cell[2] * np.array([np.cos(np.radians(cell[4])), 0.0, np.sin(np.radians(cell[4]))])
            s2 = (np.linalg.norm(H @ np.linalg.inv(a).T, axis=1) / 2) ** 2
            e = 800.0 * scale * s2 / np.log(10.0)       # the factor's decimal exponent
            assert not np.any((e > 125) & (e < 156))
            want = e > 140
            assert 0 < want.sum() < len(H)
    if kind == synth.MAGNETIC:
        want[np.all(H == 0, axis=1)] = False
    say(f"Bragg points of one configuration kind={kind} order={order} {bad}")
    I = gpu_intensity(m).reshape(m.count)[::3, ::4, ::5].reshape(-1)
    assert np.array_equal(np.isnan(I), want)
    assert not np.any(I[~want])


@pytest.mark.parametrize("M", [1, 3, 9])
@pytest.mark.parametrize("b,amp,norm", [(1e-18, 1e3, 1e4), (1e-25, 1e10, 1.0), (3e17, 0.5, 1e10), (1e22, 1e-5, 1e25), (0.0, 1.0, 1.0)])
def test_one_site_tiles_with_small_and_large_weights(M, b, amp, norm):
    """A site weight whose square, or its product with the norm or an amplitude, leaves the normal
    float32 range though the intensities do not."""
    m = synth.random_model(3500 + M, n=(20, 24, 40), S=1, M=M, order=0, with_disp=False)
    m.b[:] = b
    m.norm_N = norm
    m.occ = (m.occ - 0.5) * np.float32(amp)
    m.g0, m.count = (-5, -6, -45), (9, 11, 83)
    say(f"one site b={b} M={M}")
    sampled_parity(m, most=1500)


# ------------------------------------------------------------------ rows of a prime length, planes past the LDS
@pytest.mark.parametrize("n,kind,order,M", [((2, 188, 205), synth.NUCLEAR, 1, 1), ((1, 141, 246), synth.NUCLEAR, 0, 2), ((2, 185, 188), synth.MAGNETIC, 0, 1),
                                            ((1, 235, 235), synth.NUCLEAR, 1, 1), ((3, 244, 208), synth.NUCLEAR, 0, 1), ((1, 240, 253), synth.MAGNETIC, 0, 2)])
def test_plane_rows_route_of_prime_edges(n, kind, order, M):
    """Rows along axis 3 per block, then axis 2 in place, where one of those edges or both have a
    prime factor from 17 to 47, odd and even numbers of rows (244 = 61 x 4: Stockham rows)."""
    m = synth.random_model(3600 + n[1] + n[2], n=n, S=1, M=M, order=order, kind=kind, with_disp=order > 0, sigma=0.03,
                           cell=None if kind == synth.NUCLEAR else [6.0, 7.0, 8.0, 90.0, 90.0, 90.0])
    m.g0, m.count = (-2, -9, -9), (5, 19, 19)
    say(f"row route of prime edges n={n} kind={kind}")
    sampled_parity(m, order if order and kind == synth.NUCLEAR else None, 1500)


@pytest.mark.parametrize("M", [1, 2, 3, 20])
@pytest.mark.parametrize("b", [np.inf, np.nan, 1e160])
def test_one_site_tiles_with_a_weight_past_float32(M, b):
    """No finite value anywhere, in ensembles none at all."""
    m = synth.random_model(3700 + M, n=(6, 5, 18), S=1, M=M, order=0, with_disp=False)
    m.b[:] = b
    m.g0, m.count = (-5, -6, -20), (9, 11, 41)
    say(f"one site b={b} M={M}")
    I = gpu_intensity(m)
    assert not np.any(np.isfinite(I)) and (M < 3 or np.all(np.isnan(I)))


@pytest.mark.parametrize("n,g0,count", [((6, 7, 12), (-12, -14, -24), (24, 28, 48)), ((6, 7, 12), (-12, -14, -24), (25, 29, 49)),
                                        ((5, 6, 20), (-10, -12, -60), (21, 25, 120)), ((5, 6, 20), (-10, -12, -40), (21, 25, 81)),
                                        ((8, 7, 9), (-60, -60, -72), (121, 121, 145)), ((31, 30, 31), (-93, -93, -93), (187, 187, 187)),
                                        ((40, 41, 6), (-41, -42, 1), (83, 85, 7)), ((9, 9, 24), (-72, -72, -48), (145, 145, 96))])
@pytest.mark.parametrize("M", [1, 2])
def test_one_site_tiles_or_voxels(n, g0, count, M):
    """Both sides of the rule between the tiled rows and the direct form: few and many repeats along
    axis 3, rows on 16 bytes and not, small and large boxes, rows of few values."""
    m = synth.random_model(3800 + sum(n) + M, n=n, S=1, M=M, order=0, with_disp=False)
    m.g0, m.count = g0, count
    say(f"one site n={n} M={M} box={g0}+{count}")
    sampled_parity(m)


@pytest.mark.parametrize("n,g0,count", [((20, 26, 14), (-40, -52, -2), (81, 105, 5)), ((20, 26, 14), (-40, -52, 3), (80, 105, 17)),
                                        ((12, 13, 40), (-12, -13, -40), (25, 27, 81)), ((25, 24, 24), (-25, -24, -48), (51, 49, 97)),
                                        ((9, 11, 24), (-9, -22, -72), (19, 45, 145)), ((30, 31, 7), (-30, -62, -2), (61, 125, 5))])
@pytest.mark.parametrize("M,b", [(1, 1.0), (2, 1.0), (3, 1.0), (5, 1e22), (8, 1.0), (12, 1.0), (3, np.inf), (8, 1e160)])
def test_one_site_ensembles_tiles_or_voxels(n, g0, count, M, b):
    """The same for ensembles and for boxes thinner than the supercell, with a weight whose square
    leaves float32, and with weights past it (which leave no value)."""
    m = synth.random_model(3900 + sum(n) + M, n=n, S=1, M=M, order=0, with_disp=False)
    m.b[:] = b
    m.g0, m.count = g0, count
    if b == 1e22:
        m.norm_N = 1e25
        m.occ = (m.occ - 0.5) * np.float32(1e-5)
    say(f"one site n={n} M={M} b={b} box={g0}+{count}")
    if b in (np.inf, 1e160):
        assert np.all(np.isnan(gpu_intensity(m)))
    else:
        sampled_parity(m, most=1500)
