"""Renders begun and ended by separate calls, or forked ahead, keep their sub-chunk streams
(work on the caller's stream runs beside them) from 2^17 paths on, where a render in one
call stays on the caller's stream; the images are the same."""
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


def _extend_launches(render):
    from paper_2106_12802_amd import tracer as R
    try:
        R.profile_select(["extend"])
        R.profile_enable(True)
        render()
        return R.profile_read()["extend"][1]
    finally:
        R.profile_enable(False)
        R.profile_select(None)


# paths of the pair of jobs: 114,688; 2^17; 215,040; 2^18
@pytest.mark.parametrize("W,H,spp,streams", [(128, 128, 7, 1), (128, 128, 8, 2), (192, 160, 7, 3),
                                             (256, 128, 8, 3)])
# all resident in both ways of rendering, in one of them, in none
@pytest.mark.parametrize("chunk", [None, -100, 40_000])
def test_split_renders_keep_their_streams(mrs, W, H, spp, streams, chunk):
    import torch
    gs = mrs.GpuScene(S.cornell(2))
    total = W * H * spp
    jobs = [dict(scene=gs, W=W, H=H - 8, spp=spp, max_depth=4, seed=5),
            dict(scene=gs, W=W, H=8, spp=spp, max_depth=4, seed=6, want_aux=False)]
    ref = [mrs.render(gs, j["W"], j["H"], spp, 4, j["seed"], want_aux=j.get("want_aux", True))
           for j in jobs]
    torch.cuda.synchronize()
    if chunk is not None:
        mrs.set_tuning(chunk_paths=chunk if chunk > 0 else total + chunk)
    b = mrs.Batch(jobs)

    def split():
        b.render_begin()
        b.render_end()

    def forked_split():
        b.render_fork()
        split()

    def forked():
        b.render_fork()
        b.render()

    ways = [(b.render, 1), (split, streams), (forked_split, streams), (forked, streams)]
    for _ in range(2):
        for way, k in ways:
            for pair in b.outputs:
                for t in pair:
                    if t is not None:
                        t.fill_(-1.0)
            n = _extend_launches(way)
            assert chunk is not None or n == k, way
            torch.cuda.synchronize()
            for got, want in zip(b.outputs, ref):
                assert torch.equal(got[0], want[0])
                assert want[1] is None or torch.equal(got[1], want[1])
    b.close()
