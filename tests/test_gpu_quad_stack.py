"""Four lanes per ray share one stack: 64 entries in LDS, the rest in memory.  A ladder of
boxes whose traversal needs more of them than that gives bitwise the results of one lane
per ray on every route, camera and shadow rays alike."""
import sys

import numpy as np
import pytest

from mrs_inputs import scenes as S

sys.path.insert(0, __file__.rsplit("/", 1)[0])
from test_ploc_model import LEAF, _half_area, _morton_order, cluster, layout  # noqa: E402

LDS_ENTRIES = 64


def _ladder(levels=28):
    """Triangles across the z axis: one, then on each level a larger one and two larger ones
    close together.  The clustering joins the two with each other and the ladder so far with
    the one, so a four-wide node holds the ladder so far and three triangles, and a ray
    along z from in front of the first one descends to it with the others on its stack.
    Behind the camera a wall whose light comes through the ladder."""
    b = S._Builder()
    grey = b.material(S.LAMBERT, (0.5, 0.5, 0.5))
    base = np.array([[-1.0, -1.0, 0.0], [1.0, -1.0, 0.0], [0.0, 2.0, 0.0]])
    tris, w, z = [base * 20.0], 20.0, 0.0
    for _ in range(levels):
        for grow, dz in ((1.04, 0.01), (1.04, 0.01), (1.0, 0.001)):
            w, z = w * grow, z + dz
            tris.append(base * w + np.array([0.0, 0.0, z]))
    b.add_tris(tris, grey)
    b.add_tris([base[::-1] * 3000.0 + np.array([0.0, 0.0, -10.0])], grey)
    b.add_light((-2.0, -2.0, 5.0), (0.0, 4.0, 0.0), (4.0, 0.0, 0.0), (9.0, 9.0, 9.0))
    return b.build((0.3, 0.4, 0.5), S.Camera((0, 0, -5), (0, 0, 0)), "ladder")


def _entries(tri, o, d):
    """Stack entries of the nearest-first walk of ray o + t d down to its first leaf."""
    children, root, _, _ = cluster(tri)
    t3 = tri[_morton_order(tri)]
    box = {}

    def bounds(r):
        if r not in box:
            if r & LEAF:
                v = t3[r & ~LEAF]
                box[r] = (v.min(0), v.max(0))
            else:
                (l, h), (l2, h2) = (bounds(int(c)) for c in children[r])
                box[r] = (np.minimum(l, l2), np.maximum(h, h2))
        return box[r]

    def entry(r):  # None: missed
        lo, hi = bounds(r)
        t = np.stack([(lo - o) / d, (hi - o) / d])
        near, far = max(t.min(0).max(), 0.0), t.max(0).min()
        return near if near <= far else None

    deepest, sp, node = 0, 0, root
    while not node & LEAF:
        c = [int(x) for x in children[node]]
        for _ in range(2):  # the child of largest area is opened, twice
            inner = [i for i in range(len(c)) if not c[i] & LEAF]
            if inner:
                i = max(inner, key=lambda k: _half_area(*bounds(c[k])))
                c[i:i + 1] = [int(x) for x in children[c[i]]]
        hit = sorted((r for r in c if entry(r) is not None), key=entry)
        sp += len(hit) - 1
        deepest, node = max(deepest, sp), hit[0]
    return deepest


# a camera ray, and a shadow ray from the wall
RAYS = [((0.0, 0.0, -5.0), (1e-3, 2e-3, 1.0)), ((3.0, -4.0, -9.99), (-0.1, 0.2, 1.0))]


@pytest.mark.parametrize("o,d", RAYS)
def test_the_ladder_needs_more_entries_than_lds_holds(o, d):
    tri = _ladder().vertices.astype(np.float32)
    children, root, _, _ = cluster(tri)
    assert layout(children, root, len(tri))[3] <= 64  # else the other builder takes it
    assert LDS_ENTRIES + 16 < _entries(tri, np.array(o), np.array(d)) < 128


@pytest.mark.gpu
@pytest.mark.parametrize("W,H,spp", [(1, 1, 1), (33, 17, 2), (300, 200, 2)])
def test_deep_stacks_on_every_route(W, H, spp):
    """One path, waves that are not full, more paths than one launch takes whole."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2106_12802_amd as mrs
    old = mrs.get_tuning()
    try:
        mrs.set_tuning(bvh_leaf_max=1)
        gs = mrs.GpuScene(_ladder())
        assert gs.bvh_builder == "ploc"

        def render(**tuning):
            mrs.set_tuning(**old)
            mrs.set_tuning(**tuning)
            mrs.counters(reset=True)
            out = mrs.render(gs, W, H, spp, 4, 7)
            torch.cuda.synchronize()
            return out, mrs.counters(reset=True)

        ref, n = render(schedule=1)
        assert n["overflows"] == 0 and torch.isfinite(ref[0]).all()
        for tuning in ({}, dict(tail_bounce=1), dict(tail_bounce=65), dict(wave_extend=0),
                       dict(wave_extend=0, tail_bounce=65), dict(trace_blocks=3)):
            got, m = render(**tuning)
            assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1]), tuning
            assert all(m[k] == n[k] for k in ("rays", "shadow_rays", "paths", "overflows"))
            # entries beyond LDS: on the first and the last two all rays are a quad's
            if tuning in ({}, dict(wave_extend=0), dict(trace_blocks=3)):
                assert m["spills"] > 0, tuning
    finally:
        mrs.set_tuning(**old)
