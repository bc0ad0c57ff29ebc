"""Nodes close to the most arcs and vertices that a node may have (192 and
128; a node of v struts that is covered by them has 3 (v - 2) and 2 (v - 2)),
and nodes beyond what can be meshed: stars of 40 to 64 struts whose hub grows
until its cones no longer meet in ellipses.  One lane per node, where the
pieces of a conic are finished one after another, and the wave schedule agree
on every output, and a node that cannot be meshed leaves the others whole."""

import types

import numpy as np
import pytest

from parity import result_np

pytestmark = pytest.mark.gpu


def _stars(v):
    """Stars of v struts, the hub from almost as thin as its struts to almost as long."""
    rng = np.random.default_rng(v)
    i = np.arange(v) + 0.5
    phi, th = np.arccos(1 - 2 * i / v), np.pi * (1 + 5**0.5) * i
    d = np.stack([np.cos(th) * np.sin(phi), np.sin(th) * np.sin(phi), np.cos(phi)], 1)
    pos, rad, ends, status = [], [], [], []
    for s, rho in enumerate(np.geomspace(0.02, 0.97, 23)):
        e = d + 0.06 * rng.normal(size=d.shape)
        c, first = np.array([4.0 * s, 0.0, 0.0]), s * (v + 1)
        pos += [c[None], c + e / np.linalg.norm(e, axis=1, keepdims=True)]
        rad += [[rho], rng.uniform(0.01, 0.03, v)]
        ends.append(np.stack([np.full(v, first), first + 1 + np.arange(v)], 1))
    pos, rad, ends = np.concatenate(pos), np.concatenate(rad), np.concatenate(ends)
    f = lambda a: np.ascontiguousarray(a, np.float32)  # noqa: E731
    return types.SimpleNamespace(x=f(pos[:, 0]), y=f(pos[:, 1]), z=f(pos[:, 2]), radius=f(rad),
                                 strut_a=ends[:, 0].astype(np.int32), strut_b=ends[:, 1].astype(np.int32))


@pytest.mark.parametrize("v", [40, 52, 58, 64])
def test_schedules_agree_near_the_capacities(v):
    from paper_2405_15197_amd import Mesher

    lat, out = _stars(v), []
    for thread in (False, True):
        m = Mesher(lat)
        try:
            m.set_schedule(thread)
            out.append(result_np(m.run(7)))
        finally:
            m.close()
    a, b = out
    hub = a["status"][:: v + 1]
    sizes = np.diff(a["node_off"].reshape(5, -1))[:2, :: v + 1]
    print(f"{v} struts: status {sorted(set(hub.tolist()))}, at most {sizes[0].max()} vertices and {sizes[1].max()} arcs",
          flush=True)
    assert (hub != 0).any() and (hub == 0).any()
    assert sizes[0].max() >= 2 * (v - 2) and sizes[1].max() >= 3 * (v - 2)
    for key in ("status", "node_off", "strut_off", "vert_name", "vert_xyz", "arc_u32", "arc_f32", "tri", "mesh"):
        assert np.array_equal(a[key], b[key]), key
