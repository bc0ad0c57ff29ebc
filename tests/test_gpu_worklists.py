"""Work distribution of the node pass: every node of a list is meshed once,
whatever the list's length against the sixteen sub-lists, the tiles that nodes
are dealt in and the first ranges of the grid, and wherever in the sub-lists
the nodes handed to FP64 fall.  The lattices are copies of one small part, so
each copy must give the part's own mesh (counts, names and arcs)."""

import numpy as np
import pytest

import latgen
from test_gpu_pieces import ring

pytestmark = pytest.mark.gpu


def copies(part, n, pad=0):
    """n copies of a part, each with `pad` nodes without struts after it."""
    m = part.n_nodes + pad
    at = (np.arange(n)[:, None] * m + np.arange(part.n_nodes)[None]).ravel()
    xyz = np.zeros((n * m, 3), np.float32)
    xyz[at] = np.tile(part.xyz64().astype(np.float32), (n, 1))
    radius = np.full(n * m, 0.1, np.float32)
    radius[at] = np.tile(part.radius, n)
    first = np.repeat(np.arange(n) * m, part.n_struts)
    return latgen.Lattice(x=xyz[:, 0].copy(), y=xyz[:, 1].copy(), z=xyz[:, 2].copy(), radius=radius,
                          strut_a=(np.tile(part.strut_a, n) + first).astype(np.int32),
                          strut_b=(np.tile(part.strut_b, n) + first).astype(np.int32))


def check(part, n, pad, k, kappa_max):
    from paper_2405_15197_amd import Mesher

    one, many = (Mesher(lat, kappa_max=kappa_max) for lat in (part, copies(part, n, pad)))
    try:
        a, b = one.run(k), many.run(k)
        for f in ("n_vertices", "n_arcs", "n_holes", "n_mesh_vertices", "n_triangles", "n_fp64_nodes"):
            assert b.totals[f] == n * a.totals[f], f
        assert b.totals["n_bad_nodes"] == n * (a.totals["n_bad_nodes"] + pad)
        assert b.totals["n_skipped_struts"] == n * a.totals["n_skipped_struts"]
        for f, axis in (("vert_name", 0), ("vert_xyz", 1), ("arc_f32", 1)):
            x, y = getattr(a, f).cpu().numpy(), getattr(b, f).cpu().numpy()
            assert np.array_equal(np.concatenate([x] * n, axis=axis), y), f
        wa, wb = one.sink(k, part.n_nodes), many.sink(k, max(many.n_nodes // 3, 1))
        assert wb[:, 0].sum() == n * wa[:, 0].sum() and wb[:, 2].sum() == n * wa[:, 2].sum()
        return b.totals
    finally:
        one.close()
        many.close()


def fan(nstrut, seed=1):
    """A centre of nstrut struts."""
    rng = np.random.default_rng(seed)
    return latgen.star(rng.normal(size=(nstrut, 3)), radius=0.02)


@pytest.mark.parametrize("n", [1, 15, 16, 17, 33, 257])
@pytest.mark.parametrize("nstrut", [3, 7, 11, 20], ids=["four_per_wave", "two_per_wave", "one_per_wave", "multi_wave"])
@pytest.mark.parametrize("kappa_max", [None, 0.0], ids=["fp32", "fp64"])
def test_short_lists(n, nstrut, kappa_max):
    print(n, nstrut, check(fan(nstrut), n, 0, 8, kappa_max), flush=True)


@pytest.mark.parametrize("n", [4095, 4097, 8200])
def test_lists_beyond_the_grid(n):
    # one centre per copy: more of them than the 4,096 blocks of a launch
    t = check(fan(9), n, 0, 6, None)
    print(n, t, flush=True)


def test_long_list_in_tiles():
    # 840,000 strut ends, four per wave: 210,000 items, above the 131,072 from
    # which a grid of 4,096 blocks is dealt tiles of sixteen
    check(fan(6), 140000, 0, 4, None)


@pytest.mark.parametrize("n", [5, 700, 3000])
def test_fp64_nodes_in_one_sub_list(n):
    # the centre of each ring (three pieces of one conic) goes to FP64; with
    # sixteen nodes per copy all of them fall into one sub-list
    part = ring(3, 0)
    t = check(part, n, 16 - part.n_nodes, 8, None)
    print(n, t, flush=True)
    assert t["n_fp64_nodes"] >= n


@pytest.mark.parametrize("n", [65536, 65537])
def test_longest_list_given_out_whole_and_shortest_grabbed(n):
    # sixteen rounds over the 4,096 waves of a launch, and one node more
    check(fan(9), n, 0, 3, None)
