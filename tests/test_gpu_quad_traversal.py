"""Small renders: four lanes per ray (quad traversal), whole paths in one launch and the
earlier path tail give bitwise the results of one lane per ray.  schedule = 1 (a queue
counter per launch) keeps one lane per ray and a launch per kernel, tail_bounce = 65
a launch per bounce."""
import numpy as np
import pytest

from mrs_inputs import scenes as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.fixture(scope="module")
def scenes():
    import paper_2106_12802_amd as mrs
    b = S._Builder()
    m = b.material(S.LAMBERT, (0.5, 0.5, 0.5))
    base = np.array([[-1.0, -1.0, 0.0], [1.0, -1.0, 0.0], [0.0, 1.0, 0.0]])
    b.add_tris([base * 1.3 ** k + np.array([0.0, 0.0, 0.01 * k]) for k in range(60)], m)
    chain = b.build((0.3, 0.4, 0.5), S.Camera((0, 0, -5), (0, 0, 0)), "chain")
    one = S._Builder()
    one.add_tris([base], one.material(S.LAMBERT, (0.5, 0.6, 0.7)))
    single = one.build((0.3, 0.4, 0.5), S.Camera((0, 0, -3), (0, 0, 0)), "single")
    made = {"box": S.cornell(2), "procedural": S.procedural_sized(11, 12_000),
            "single": single, "empty": S.env_only((0.3, 0.5, 0.7))}
    out = {k: mrs.GpuScene(v) for k, v in made.items()}
    old = mrs.get_tuning()
    try:
        mrs.set_tuning(bvh_leaf_max=1)  # a chain of 20 nodes: stacks beyond one lane's LDS
        out["chain"] = mrs.GpuScene(chain)
    finally:
        mrs.set_tuning(**old)
    return out


def _render(mrs, torch, gs, W, H, spp, depth, seed, tuning, **kw):
    old = mrs.get_tuning()
    lay = torch.full((H, W, 9), float("nan"), device="cuda")
    sq = torch.full((H, W, 3), float("nan"), device="cuda")
    mrs.counters(reset=True)
    try:
        mrs.set_tuning(**tuning)
        rgb, aux = mrs.render(gs, W, H, spp, depth, seed, out_layers=lay, out_sumsq=sq, **kw)
        torch.cuda.synchronize()
    finally:
        mrs.set_tuning(**old)
    c = mrs.counters(reset=True)
    assert c["overflows"] == 0 and c["nonfinite"] == 0
    return [rgb, aux, lay, sq], (c["rays"], c["shadow_rays"], c["paths"])


# paths: one; a wave that is not full; both sides of the lines at 2^16, 2^17, 2^18, 2^19
SIZES = [(1, 1, 1), (7, 3, 1), (33, 17, 2), (256, 256, 1), (257, 256, 1), (256, 256, 2),
         (257, 256, 2), (256, 256, 4), (257, 256, 4), (512, 256, 4), (513, 256, 4)]


@pytest.mark.parametrize("scene", ["box", "procedural"])
@pytest.mark.parametrize("W,H,spp", SIZES)
def test_small_renders_on_every_route(torch_cuda, scenes, scene, W, H, spp):
    import paper_2106_12802_amd as mrs
    gs = scenes[scene]
    kw = dict(mis=True, lens_radius=0.05, focus_dist=9.0, cam_motion=(0.1, 0.0, 0.0))
    ref, n = _render(mrs, torch_cuda, gs, W, H, spp, 6, W + H, dict(schedule=1), **kw)
    assert all(torch_cuda.isfinite(t).all() for t in ref)
    for tuning in ({}, dict(tail_bounce=65), dict(tail_bounce=1), dict(wave_extend=0),
                   dict(trace_blocks=7), dict(streams=1)):
        got, m = _render(mrs, torch_cuda, gs, W, H, spp, 6, W + H, tuning, **kw)
        assert all(torch_cuda.equal(a, b) for a, b in zip(ref, got)), tuning
        assert m == n, tuning


@pytest.mark.parametrize("scene", ["chain", "single", "empty", "box"])
@pytest.mark.parametrize("depth", [0, 1, 8])
def test_degenerate_trees_and_depths(torch_cuda, scenes, scene, depth):
    import paper_2106_12802_amd as mrs
    gs = scenes[scene]
    ref, n = _render(mrs, torch_cuda, gs, 40, 30, 3, depth, 5, dict(schedule=1))
    for tuning in ({}, dict(tail_bounce=65), dict(wave_extend=0)):
        got, m = _render(mrs, torch_cuda, gs, 40, 30, 3, depth, 5, tuning)
        assert all(torch_cuda.equal(a, b) for a, b in zip(ref, got)), tuning
        assert m == n, tuning


def test_small_batch_of_mixed_scenes(torch_cuda, scenes):
    """Jobs of several scenes in one launch of whole paths, rendered twice."""
    import paper_2106_12802_amd as mrs
    torch = torch_cuda
    jobs = [dict(scene=scenes[k], W=31, H=17, spp=s, max_depth=5, seed=9 + s)
            for k, s in (("box", 2), ("procedural", 5), ("empty", 1), ("single", 3), ("chain", 2))]
    b = mrs.Batch(jobs)
    for _ in range(2):
        b.render()
    torch.cuda.synchronize()
    for j, (rgb, aux) in zip(jobs, b.outputs):
        ref, _ = _render(mrs, torch, j["scene"], 31, 17, j["spp"], 5, j["seed"], dict(schedule=1))
        assert torch.equal(rgb, ref[0]) and torch.equal(aux, ref[1])


def test_whole_paths_under_capture(torch_cuda, scenes):
    """A captured small batch replays bitwise, with other renders between the replays."""
    import paper_2106_12802_amd as mrs
    torch = torch_cuda
    gs = scenes["procedural"]
    ref, _ = _render(mrs, torch, gs, 64, 48, 2, 5, 21, dict(schedule=1))
    b = mrs.Batch([dict(scene=gs, W=64, H=48, spp=2, max_depth=5, seed=21)])
    b.render()
    torch.cuda.synchronize()
    (rgb, aux), = b.outputs
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        b.render()
    for _ in range(3):
        rgb.fill_(-1.0)
        aux.fill_(-1.0)
        mrs.render(scenes["box"], 20, 20, 1, 3, 1)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(rgb, ref[0]) and torch.equal(aux, ref[1])
