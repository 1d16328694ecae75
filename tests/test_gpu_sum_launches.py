"""The launches of the per-pixel sums: one for each kernel class among the jobs of a batch,
whatever their order; each launch's time is recorded once."""
import pytest

from mrs_inputs import scenes as S

pytestmark = pytest.mark.gpu


@pytest.fixture
def mrs():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2106_12802_amd as mrs
    old = mrs.get_tuning()
    yield mrs
    mrs.set_tuning(**old)


# resident at once; in super-chunks that cut jobs and pixels
@pytest.mark.parametrize("chunk", [None, 5000])
def test_one_launch_per_class_for_alternating_jobs(mrs, chunk):
    """40 jobs, in turn: features at 4 spp (a thread per pixel), radiance at 33 spp (16 lanes,
    FP32) and, twice, at 1024 spp (16 lanes, FP64)."""
    import torch
    from paper_2106_12802_amd import tracer as R
    gs = mrs.GpuScene(S.cornell(2))
    jobs = []
    for i in range(40):
        spp = 1024 if i in (10, 21) else (4, 33)[i % 2]
        jobs.append(dict(scene=gs, W=9 + i % 4, H=5 + i % 3, spp=spp, max_depth=3, seed=70 + i,
                         want_aux=i % 2 == 0))
    total = sum(j["W"] * j["H"] * j["spp"] for j in jobs)
    if chunk:
        mrs.set_tuning(chunk_paths=chunk)
    b = mrs.Batch(jobs)
    try:
        R.profile_select(["accumulate"])
        R.profile_enable(True)
        b.render()
        launches = R.profile_read()["accumulate"][1]
    finally:
        R.profile_enable(False)
        R.profile_select(None)
    assert launches <= 3 * (1 if chunk is None else -(-total // 5120))
    assert chunk or launches == 3
    for j, (rgb, aux) in zip(jobs, b.outputs):
        r1, a1 = mrs.render(gs, j["W"], j["H"], j["spp"], 3, j["seed"], want_aux=j["want_aux"])
        torch.cuda.synchronize()
        assert torch.equal(rgb, r1)
        assert not j["want_aux"] or torch.equal(aux, a1)
    b.close()


def test_resolve_without_a_launch_has_no_time(mrs):
    """A render whose paths are all resident writes its outputs from the sums' kernel: counted
    as its resolve, timed as sums; one in super-chunks has a resolve launch of its own."""
    from paper_2106_12802_amd import tracer as R
    gs = mrs.GpuScene(S.cornell(2))
    got = {}
    for chunk in (mrs.get_tuning()["chunk_paths"], 1000):
        mrs.set_tuning(chunk_paths=chunk)
        try:
            R.profile_select(["accumulate", "resolve"])
            R.profile_enable(True)
            mrs.render(gs, 64, 64, 2, 3, 1)
            got[chunk] = R.profile_read()
        finally:
            R.profile_enable(False)
            R.profile_select(None)
    direct, chunked = got.values()
    assert direct["accumulate"][0] > 0.0 and direct["accumulate"][1] == 1
    assert direct["resolve"] == (0.0, 1)
    assert chunked["resolve"][0] > 0.0 and chunked["resolve"][1] == 1
