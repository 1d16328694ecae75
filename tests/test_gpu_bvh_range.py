"""Clustering of boxes beyond FP32's range: a cost of infinity is a cost, one that is not a
number is none, and a round without a merge is refused."""
import numpy as np
import pytest

from mrs_inputs import scenes as S

pytestmark = pytest.mark.gpu


@pytest.fixture
def mrs():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2106_12802_amd as mrs
    return mrs


def _scene(points):
    """A degenerate triangle at each point (its box is the point)."""
    b = S._Builder()
    b.add_tris(np.repeat(np.array(points, np.float64)[:, None], 3, 1),
               b.material(S.LAMBERT, (0.5, 0.5, 0.5)))
    return b.build((0.3, 0.4, 0.5), S.Camera((0, 0, -3), (0, 0, 0)), "points")


def test_a_pair_of_infinite_cost_merges(mrs):
    """In Morton order 0, 1, 2; 0 + 1 and 1 + 2 are infinitely long and flat (infinity times
    zero), 0 + 2 is merely too large: they merge, then all three."""
    gs = mrs.GpuScene(_scene([(-3e38, 0, 0), (3e38, 0, 1e30), (-3e38, 1e30, 1e30)]))
    assert gs.bvh_builder == "ploc"


@pytest.mark.parametrize("n", [2, 3, 8])
def test_no_pair_with_a_cost_is_refused(mrs, n):
    """Points at the two ends of the x axis, in turn: those of an end merge, the ends' union
    is infinitely long and flat."""
    from paper_2106_12802_amd._lib import MrsError
    pts = [((-3e38, 3e38)[i % 2], 0.0, 0.0) for i in range(n)]
    with pytest.raises(MrsError, match="merged nothing"):
        mrs.GpuScene(_scene(pts))
