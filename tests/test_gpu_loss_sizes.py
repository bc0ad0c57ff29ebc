"""The mesh loss at both sizes of a node's room in LDS, each for nodes that fit it
and nodes that pass over their triangles again, and beyond the passes; against
the same triangles in FP64, with the tolerance of test_gpu_loss.py."""

import pytest

import latgen
import test_gpu_loss

pytestmark = pytest.mark.gpu

# more nodes than the chip holds at the larger room; fewer go to it at any k
CASES = [("knn15_9", lambda: latgen.knn(15, 9, ("uniform", 0.04, 0.12), seed=3), 64),  # small: most fit
         ("bcc12", lambda: latgen.bcc(12, ("uniform", 0.05, 0.12), 0.05, seed=2), 190),  # large: they fit
         ("bcc12", lambda: latgen.bcc(12, ("uniform", 0.05, 0.12), 0.05, seed=2), 300),  # small: three passes
         ("knn15_9", lambda: latgen.knn(15, 9, ("uniform", 0.04, 0.12), seed=3), 130),  # large: some of two passes
         ("knn9_9", lambda: latgen.knn(9, 9, ("uniform", 0.04, 0.12), seed=3), 100),  # few nodes: large
         ("knn9_9", lambda: latgen.knn(9, 9, ("uniform", 0.04, 0.12), seed=3), 400)]  # large: and beyond the passes


@pytest.mark.parametrize("name,make,k", CASES, ids=[f"{c[0]}_k{c[2]}" for c in CASES])
def test_loss_gradient_by_room(name, make, k):
    test_gpu_loss.test_loss_gradient(name, make, k, (0.7, -1.3, 0.4))


def test_a_retriangulated_mesh_has_its_own_resolution():
    """The room follows the mesh's resolution: the gradient is that of a mesh made at it."""
    import torch

    from paper_2405_15197_amd import Mesher

    m = Mesher(latgen.bcc(12, ("uniform", 0.05, 0.12), 0.05, seed=2))
    try:
        at = {k: m.run(k) for k in (190, 8)}
        again = m.retriangulate(190)
        same = m.loss(again, (0.7, -1.3, 0.4))[1]
        m.run(190)
        assert torch.equal(again.tri, at[190].tri) and torch.equal(same, m.loss(at[190], (0.7, -1.3, 0.4))[1])
    finally:
        m.close()
