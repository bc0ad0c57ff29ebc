"""The adjoint at the free end of a strut, against the same points in FP64: its
hole is the whole circle where the cone touches the node's sphere, and the hole's
centre lies on the strut's axis however small the difference of the radii is."""

import math

import numpy as np
import pytest

import latgen

pytestmark = pytest.mark.gpu

EPS = 2.0**-24


def _end(torch, c, rho, far, r_far, up, k):
    """Mesh vertices of a node with one strut: the circle's points, then the centre of its hole."""
    d = far - c
    length = d.square().sum().sqrt()
    e, sig = d / length, (rho - r_far) / length
    kap = (1 - sig * sig).sqrt()
    es = e if up else -e
    axis = torch.eye(3, dtype=torch.float64)[es.detach().abs().argmin()]
    r = torch.linalg.cross(es, axis)
    r = r / r.square().sum().sqrt()
    q = torch.linalg.cross(es, r)
    t = 2 * math.pi * torch.arange(k, dtype=torch.float64)[:, None] / k
    ring = rho * sig * e + rho * kap * (q * t.sin() + r * t.cos())
    return c + torch.cat([ring, -rho * e[None]])


@pytest.mark.parametrize("alike", [0.3, 1e-2, 1e-3, 1e-5, 0.0])
@pytest.mark.parametrize("k", [3, 10, 150])
def test_free_ends(k, alike):
    import torch

    from paper_2405_15197_amd import Mesher

    lat = latgen.star([(0.7, 0.4, -0.5)], radii=[0.1, 0.1 * (1 - alike)])
    m = Mesher(lat)
    try:
        got = m.run(k, meta=False)
        x = torch.tensor(np.stack([lat.x, lat.y, lat.z], 1), dtype=torch.float64).requires_grad_(True)
        rad = torch.tensor(lat.radius, dtype=torch.float64).requires_grad_(True)
        want = torch.cat([_end(torch, x[i], rad[i], x[1 - i], rad[1 - i], i == 0, k) for i in range(2)])
        assert (got.mesh_xyz.cpu().double() - want).abs().max() < 1e-6
        lam = torch.randn(want.shape, generator=torch.Generator().manual_seed(k))
        gx, gr = m.backward(lam.cuda())
        wx, wr = torch.autograd.grad((want * lam.double()).sum(), (x, rad))
        # the sums' terms are at most |lambda| long, and pass some twenty roundings each
        tol = 32 * EPS * lam.double().norm(dim=1).sum()
        err = max((gx.cpu() - wx).abs().max(), (gr.cpu() - wr).abs().max())
        print(f"k {k}, radii alike to {alike}: error {float(err):.2e}, tolerance {float(tol):.2e}", flush=True)
        assert err <= tol
    finally:
        m.close()
