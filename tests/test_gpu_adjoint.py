"""The adjoint at the edges of its work split, against the FP64 oracle's
central differences: whole circles (one strut, equal and unequal ends), two
struts, the most struts and the most arcs of one wave, one strut more, and a
node whose arcs take several turns of the wave (its loop table has 16-bit
entries).  Tolerance as in the other gradient tests: FP32 arithmetic through
the tie solves, 1e-3 |g| + 1e-4 max|g|."""

import numpy as np
import pytest

import latgen
import oracle

pytestmark = pytest.mark.gpu

W3 = [(1.0, 0.0, 0.0), (0.0, 1.0, 0.0), (0.0, 0.0, 1.0)]


def _dirs(n):
    i = np.arange(n) + 0.5
    phi = np.arccos(1 - 2 * i / n)
    th = np.pi * (1 + 5**0.5) * i + 0.2 * np.sin(7 * i)
    return np.stack([np.cos(th) * np.sin(phi), np.sin(th) * np.sin(phi), np.cos(phi)], 1)


def _star(n):
    rng = np.random.default_rng(n)
    return latgen.star(_dirs(n) * rng.uniform(0.8, 1.2, size=(n, 1)),
                       radii=np.r_[0.08, rng.uniform(0.04, 0.07, size=n)])


CASES = {
    "capsule": lambda: latgen.star([(1.0, 0.2, 0.1)], radius=0.1),
    "cone": lambda: latgen.star([(1.0, 0.2, 0.1)], radii=[0.1, 0.06]),
    "bent": lambda: latgen.star([(1.0, 0.1, 0.0), (0.2, 1.0, 0.3)], radii=[0.1, 0.07, 0.08]),
    "star12": lambda: _star(12),
    "star16": lambda: _star(16),
    "star17": lambda: _star(17),
    "star40": lambda: _star(40),
}


@pytest.mark.parametrize("name", CASES)
def test_adjoint_matches_oracle(name):
    from paper_2405_15197_amd import Mesher

    lat, k = CASES[name](), 9
    assert (oracle.run(lat, k).status == 0).all()
    params = [(n, c) for n in sorted({0, 1, lat.n_nodes - 1}) for c in range(4)]
    G, ok = oracle.fd_gradient(lat, k, params, weights=W3)
    M = Mesher(lat)
    try:
        r = M.run(k, meta=False)
        for wi, w in enumerate(W3):
            gx, gr = M.backward(M.loss(r, w)[1])
            gx, gr = gx.cpu().numpy().astype(np.float64), gr.cpu().numpy().astype(np.float64)
            g = np.array([gx[n, c] if c < 3 else gr[n] for n, c in params])[ok]
            want = G[:, wi][ok]
            err, tol = np.abs(g - want), 1e-3 * np.abs(want) + 1e-4 * np.abs(want).max()
            assert (err <= tol).all(), (wi, (err / tol).max(), g, want)
    finally:
        M.close()
