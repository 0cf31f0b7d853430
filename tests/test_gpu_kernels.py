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
    assert_parity(I[tuple((G - np.asarray(m.g0)).T)], O.intensity(m, G, order))


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
