"""The BVH build at the sizes where its kernels change: the rounds that one block
finishes by itself (up to 4096 clusters), the tiles of the sort (1024 keys) and of
the compaction (256 clusters; 8 x 256 above 524,288), and the collapse's levels."""
import numpy as np
import pytest

from mrs_inputs import scenes as S
from test_gpu_tracer import _check_bvh4, _check_lbvh

pytestmark = pytest.mark.gpu


@pytest.fixture
def mrs():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2106_12802_amd as mrs
    old = mrs.get_tuning()
    yield mrs
    mrs.set_tuning(**old)


@pytest.mark.parametrize("n", [2, 3, 255, 1024, 1025, 4095, 4096, 4097, 9001])
def test_clustered_tree_at_the_edges(mrs, n):
    scene = S.random_soup(n, n, spread=2.0)
    gs = mrs.GpuScene(scene)
    assert gs.bvh_builder == "ploc"
    _check_lbvh(gs, scene)
    _check_bvh4(gs, scene)


@pytest.mark.parametrize("n", [4097, 70_001, 530_000])
def test_both_builders_hit_the_same(mrs, n):
    scene = S.random_soup(3, n, spread=8.0)
    o, d = S.random_rays(4, 3000, spread=8.0)
    hits = []
    for b in ("lbvh", "ploc"):
        mrs.set_tuning(bvh_builder=b)
        gs = mrs.GpuScene(scene)
        assert gs.bvh_builder == b
        leaf = gs.bvh()[1]
        assert np.array_equal(np.sort(leaf), np.arange(n))
        hits.append(gs.closest_hit(o, d))
        gs.close()
    for x, y in zip(*hits):
        assert np.array_equal(x, y)


def test_a_rebuilt_scene_gives_the_same_tree(mrs):
    """The order in which merges are counted differs between runs; the tree does not."""
    scene = S.random_soup(8, 12_345, spread=4.0)
    a, b = mrs.GpuScene(scene), mrs.GpuScene(scene)
    for x, y in zip(a.bvh()[:3], b.bvh()[:3]):
        assert np.array_equal(x, y)
    # as words: an absent child's reference is a NaN
    assert np.array_equal(a.bvh4()[0].view(np.uint32), b.bvh4()[0].view(np.uint32))
