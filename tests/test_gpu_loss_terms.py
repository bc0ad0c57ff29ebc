"""Area and volume of long thin band triangles (struts much longer than their
segments) against the same triangles in FP64.

A triangle's area comes from the product of its edge and of a side that starts
at it: each component of that product is rounded a few times, at most EPS of
|edge| |side| each, of either sign, so that they add up as square roots over the
triangles; its square root's own rounding, at most EPS, may lean to one side.
The volume's products are of positions instead."""

import numpy as np
import pytest

import latgen

pytestmark = pytest.mark.gpu

EPS = 2.0**-24


def _star(v, length, seed):
    d = np.random.default_rng(seed).normal(size=(v, 3))
    return latgen.star(d, length=length, radii=np.r_[0.02, np.full(v, 0.015)])


@pytest.mark.parametrize("v,length,k", [(1, 1.0, 1500), (2, 3.0, 400), (5, 1.0, 700), (5, 6.0, 100), (12, 4.0, 30)])
def test_terms_of_thin_triangles(v, length, k):
    from paper_2405_15197_amd import Mesher

    off, size = np.zeros(2), np.zeros(2)
    for seed in range(6):
        m = Mesher(_star(v, length, seed))
        try:
            r = m.run(k, meta=False)
            got = m.loss(r, (0.0, 0.0, 0.0))[0].cpu().numpy()
            p = r.mesh_xyz.double()[r.tri.long()]
            a, b = p[:, 1] - p[:, 0], p[:, 2] - p[:, 0]
            area = a.cross(b, dim=1).norm(dim=1) / 2
            six = (p[:, 0] * p[:, 1].cross(p[:, 2], dim=1)).sum(1)
            edge, far = a.norm(dim=1) * b.norm(dim=1) / 2, p.norm(dim=2).prod(dim=1) / 6
            off += [(got[0] - area.sum().item()) ** 2, (got[1] - six.sum().item() / 6) ** 2]
            size += [(2 * area.sum().item() + 4 * edge.square().sum().item() ** 0.5) ** 2,
                     (2 * six.abs().sum().item() / 6 + 4 * far.square().sum().item() ** 0.5) ** 2]
        finally:
            m.close()
    print(f"{v} struts of {length}, k = {k}: area {(off[0] / size[0]) ** 0.5 / EPS:.2f}, volume "
          f"{(off[1] / size[1]) ** 0.5 / EPS:.2f} of the tolerance", flush=True)
    assert (off <= EPS**2 * size).all()
