"""The adjoint where two struts run on almost in line: the axis of their seam
ellipse comes from a small difference, and only the axis that the forward pass
took, which its points refer to, gives the gradient to rounding.

Tolerance: a gradient is a sum of the vertices' lambda times derivatives of at
most about 1; a term passes some tens of roundings of either sign, at most EPS
each, which add up as square roots: 6 EPS of the sum of all |lambda|, in the
2-norm over nodes and lattices.  Through the axis, points within the node's
radius of its centre turn by up to 1 / |gam| (half the angle) as a strut of
length 1 does: the record's conics, rounded to EPS, add radius / |gam| to that."""

import numpy as np
import pytest

import latgen
import oracle

pytestmark = pytest.mark.gpu

EPS = 2.0**-24


def _bent(angle, seed):
    """A node with two struts bent by `angle` and two or three across."""
    rng = np.random.default_rng(seed)
    r, _ = np.linalg.qr(rng.normal(size=(3, 3)))
    d = [[1.0, 0.0, 0.0], [-np.cos(angle), np.sin(angle), 0.0], [0.2, 0.3, 1.0], [-0.1, 1.0, -0.2], [0.1, -0.9, -0.8]]
    d = np.array(d[: 4 + seed % 2]) @ r
    lat = latgen.star(d, radii=0.1 * (1 + 0.05 * rng.uniform(-1, 1, len(d) + 1)))
    for x, at in zip((lat.x, lat.y, lat.z), (7, 3, 5)):  # where lambda is much the same at all vertices
        x += np.float32(at)
    return lat


@pytest.mark.parametrize("angle", [2.2e-4, 3e-4, 1e-3, 1e-2, 0.1])
def test_gradient_of_bent_struts(angle):
    from paper_2405_15197_amd import Mesher

    off = size = 0.0
    for seed in range(12):
        lat = _bent(angle, seed)
        params = [(n, c) for n in range(3) for c in range(3)]
        want, ok = oracle.fd_gradient(lat, 12, params, weights=(0.0, 0.0, 1.0))
        if not ok.all():
            continue
        m = Mesher(lat)
        try:
            r = m.run(12, meta=False)
            gx = m.backward(2 * r.mesh_xyz)[0].cpu().numpy().astype(np.float64)
            lam = 2 * np.linalg.norm(r.mesh_xyz.cpu().numpy().astype(np.float64), axis=1)
            off += sum((gx[n, c] - g) ** 2 for (n, c), g in zip(params, want))
            size += len(params) * lam.sum() ** 2 / lat.n_nodes**2
        finally:
            m.close()
    assert size > 0
    print(f"angle {angle:g}: {(off / size) ** 0.5 / EPS:.2f} EPS", flush=True)
    assert off**0.5 <= 6 * EPS * (1 + 0.1 / (angle / 2)) * size**0.5
