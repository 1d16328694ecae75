"""The collapse to four-wide nodes opens, twice, the child of largest surface area; areas of
nearly equal boxes are compared in one order of roundings, so that the tree is the one that
the binary tree's boxes give."""
import numpy as np
import pytest

from mrs_inputs import scenes as S

pytestmark = pytest.mark.gpu
LEAF = 1 << 31


def _half_areas(lo, hi):
    """fma(dx, dz, fma(dx, dy, dy dz)) in float32 (a float64 holds each product)."""
    dx, dy, dz = np.moveaxis((hi - lo).astype(np.float32).astype(np.float64), -1, 0)
    inner = (dx * dy + (dy * dz).astype(np.float32)).astype(np.float32)
    return (dx * dz + inner).astype(np.float32)


def _greedy_children(nodes, leaf_max):
    """Child references of the four-wide nodes in binary-node order."""
    words = nodes.view(np.uint32)
    area = np.stack([_half_areas(nodes[:, s:s + 3], nodes[:, s + 3:s + 6]) for s in (0, 6)], -1)

    def count(ref):
        return 1 if ref & LEAF else int(words[ref, 15]) - int(words[ref, 14]) + 1

    def pair(node):
        return [(int(words[node, 12 + s]), area[node, s]) for s in (0, 1)]

    made, todo = {}, [0]
    while todo:
        node = todo.pop()
        kids = pair(node)
        for _ in range(2):
            big = [k for k, (r, _) in enumerate(kids) if count(r) > leaf_max]
            if big:
                k = max(big, key=lambda i: (kids[i][1], -i))
                kids[k:k + 1] = pair(kids[k][0])
        made[node] = [r for r, _ in kids]
        todo += [r for r, _ in kids if count(r) > leaf_max]
    return made, count


@pytest.mark.parametrize("seed,tris,leaf_max", [(3, 60_000, 1), (11, 12_000, 3), (2, 700, 4)])
def test_the_larger_child_is_opened(seed, tris, leaf_max):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2106_12802_amd as mrs
    old = mrs.get_tuning()
    try:
        mrs.set_tuning(bvh_leaf_max=leaf_max)
        gs = mrs.GpuScene(S.procedural_sized(seed, tris))
    finally:
        mrs.set_tuning(**old)
    nodes = gs.bvh()[0]
    made, count = _greedy_children(nodes, leaf_max)
    number = {b: i for i, b in enumerate(sorted(made))}
    words = nodes.view(np.uint32)
    want = np.full((len(made), 4), 0xFFFFFFFF, np.uint32)
    for b, i in number.items():
        for k, r in enumerate(made[b]):
            if count(r) > leaf_max:
                want[i, k] = number[r]
            else:
                first = r & ~LEAF if r & LEAF else int(words[r, 14])
                want[i, k] = LEAF | (count(r) - 1) << 24 | first
    assert np.array_equal(gs.bvh4()[0].view(np.uint32)[:, 24:28], want)
