"""Conics that are kept in several pieces: the seam of two opposite, widening
struts, cut by a ring of n struts in its plane into n arcs, against the FP64
oracle.  FP32 holds two pieces (a third sends the node to FP64), FP64 four (a
fifth flags the node); the arcs of one conic come out in the order of their
smaller end names and share the numbering of the vertices that they own."""

import numpy as np
import pytest

import latgen
import oracle
from parity import compare, gpu_result

pytestmark = pytest.mark.gpu

LM_NODE_CAPACITY = 128


def ring(n, seed):
    rng = np.random.default_rng(seed)
    a = 2 * np.pi * np.arange(n) / n + rng.uniform(-0.05, 0.05, n)
    d = np.concatenate([[[0, 0, 1.0], [0, 0, -1.0]],
                        np.stack([np.cos(a), np.sin(a), rng.uniform(-0.05, 0.05, n)], 1)])
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    turn, _ = np.linalg.qr(rng.normal(size=(3, 3)))
    xyz = np.concatenate([np.zeros((1, 3)), (d * np.r_[1.0, 1.0, np.full(n, 0.15)][:, None]) @ turn.T])
    radii = np.r_[0.1, 0.5, 0.51, np.full(n, 0.02)]
    # the ring's struts in any place among the labels
    order = rng.permutation(n + 2)
    return latgen.lattice_from_arrays(xyz, radii, [(0, i + 1) for i in order], name=f"ring{n}")


@pytest.mark.parametrize("kappa_max", [None, 0.0], ids=["fp32", "fp64"])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 5])
def test_pieces_of_one_conic(n, kappa_max):
    for seed in range(4):
        lat = ring(n, seed)
        R = oracle.run(lat, 16)
        assert R.status[0] == 0
        arcs = np.asarray(R.arc_int)[: int(R.ne[0])]
        most = np.unique(arcs[:, :2], axis=0, return_counts=True)[1].max()
        assert most == n or n == 5
        G = gpu_result(lat, 16, kappa_max=kappa_max)
        print(f"ring {n} seed {seed}: {len(arcs)} arcs, fp64 nodes {G['totals']['n_fp64_nodes']}", flush=True)
        if most > 4:
            assert G["status"][0] & LM_NODE_CAPACITY
            continue
        assert G["status"][0] == 0
        if most > 2:
            assert G["totals"]["n_fp64_nodes"] > 0
        st = compare(lat, 16, R=R, G=G)
        assert st["stable"] == lat.n_nodes
