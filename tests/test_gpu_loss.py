"""The mesh loss and its gradient against the same triangles in FP64 (torch):
bands of fewer and of more triangles than a wave has lanes, nodes whose
vertices take one pass over the LDS, several, or the path beyond them."""

import numpy as np
import pytest

import latgen

pytestmark = pytest.mark.gpu

EPS = 2.0**-24


def _star(v):
    rng = np.random.default_rng(v)
    d = rng.normal(size=(v, 3))
    return latgen.star(d, radii=np.r_[0.02, rng.uniform(0.01, 0.03, v)])


CASES = [("star5", lambda: _star(5), k) for k in (3, 16, 64, 150)]
CASES += [("star12", lambda: _star(12), k) for k in (16, 70, 200, 700)]
CASES += [("star40", lambda: _star(40), k) for k in (8, 40)]
CASES += [("capsule", lambda: latgen.star([(1.0, 0.0, 0.0)], radius=0.1), k) for k in (5, 33, 300)]
CASES += [("bcc3", lambda: latgen.bcc(3, ("uniform", 0.05, 0.12), 0.05, seed=2), 24),
          ("knn4_9", lambda: latgen.knn(4, 9, ("uniform", 0.04, 0.12), seed=3), 12)]


@pytest.mark.parametrize("weights", [(1.0, 0.0, 0.0), (0.7, -1.3, 0.4)], ids=["area", "all"])
@pytest.mark.parametrize("name,make,k", CASES, ids=[f"{c[0]}_k{c[2]}" for c in CASES])
def test_loss_gradient(name, make, k, weights):
    import torch

    from paper_2405_15197_amd import Mesher

    M = Mesher(make())
    try:
        r = M.run(k)
        terms, dl = M.loss(r, weights)
        again = M.loss(r, weights)[1]
        assert torch.equal(dl, again)
        wa, wv, ws = weights
        x = r.mesh_xyz.double()
        t = r.tri.long()
        p = x[t]
        u, v = p[:, 1] - p[:, 0], p[:, 2] - p[:, 0]
        nn = torch.linalg.cross(u, v)
        nl = nn.norm(dim=1)
        area, vol = 0.5 * nl.sum(), (p[:, 0] * torch.linalg.cross(p[:, 1], p[:, 2])).sum() / 6
        sq = x.square().sum()
        got = terms.cpu().numpy()
        # FP32 terms per triangle, summed in FP64
        scale = p.norm(dim=2).prod(dim=1).sum().item()
        assert abs(got[0] - area.item()) <= 8 * EPS * (u.norm(dim=1) * v.norm(dim=1)).sum().item()
        assert abs(got[1] - vol.item()) <= 8 * EPS * scale
        assert abs(got[2] - sq.item()) <= 1e-12 * sq.item()
        n = nn / nl.clamp(min=1e-300)[:, None]
        want = 2 * ws * x
        tol = 4 * EPS * want.norm(dim=1)
        size = torch.zeros_like(tol)
        count = torch.zeros_like(tol)
        # rounding of the normal, in units of its own length
        turn = torch.where(nl > 0, 4 * EPS * u.norm(dim=1) * v.norm(dim=1) / nl.clamp(min=1e-300), 1.0).clamp(max=2.0)
        for c in range(3):
            e = p[:, (c + 2) % 3] - p[:, (c + 1) % 3]
            other = torch.linalg.cross(p[:, (c + 1) % 3], p[:, (c + 2) % 3])
            g = 0.5 * wa * torch.linalg.cross(n, e) + wv / 6 * other
            want = want.index_add(0, t[:, c], g)
            off = abs(wa) * 0.5 * e.norm(dim=1) * (2 * turn + 8 * EPS)
            off += abs(wv) / 6 * 4 * EPS * p[:, (c + 1) % 3].norm(dim=1) * p[:, (c + 2) % 3].norm(dim=1)
            tol.index_add_(0, t[:, c], off)
            size.index_add_(0, t[:, c], g.norm(dim=1))
            count.index_add_(0, t[:, c], torch.ones_like(off))
        tol += EPS * count * size  # the sum's own rounding
        err = (dl.double() - want).norm(dim=1)
        most = int(torch.bincount(torch.bucketize(torch.arange(len(x), device=x.device), r.node_off[3][1:], right=True)).max())
        print(f"{name} k={k}: {len(x)} vertices, at most {most} at a node, worst {float((err / tol).max()):.3g} of tolerance",
              flush=True)
        assert (err <= tol).all()
    finally:
        M.close()
