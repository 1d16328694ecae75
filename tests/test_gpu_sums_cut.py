"""Pixels whose samples lie in two sub-chunks that are traced concurrently: each kernel of
the per-pixel sums, straight to the outputs and through memory, equals one stream."""
import pytest

from mrs_inputs import scenes as S

pytestmark = pytest.mark.gpu


# a thread per pixel (7 spp; 31 and radiance alone), 16 lanes per pixel (17, 31 and 40)
@pytest.mark.parametrize("spp,aux,layers", [(7, True, True), (17, True, True), (31, False, False),
                                            (31, False, True), (40, False, False),
                                            (40, True, False)])
@pytest.mark.parametrize("fp64", [0, 1])
def test_pixels_cut_by_concurrent_sub_chunks(spp, aux, layers, fp64):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2106_12802_amd as mrs
    gs = mrs.GpuScene(S.cornell(2))
    H = 101
    W = 600_000 // spp // H
    total = W * H * spp
    old = mrs.get_tuning()

    def outputs(**tuning):
        mrs.set_tuning(**old)
        mrs.set_tuning(**tuning)
        sq = torch.full((H, W, 3), float("nan"), device="cuda")
        lay = torch.full((H, W, 9), float("nan"), device="cuda") if layers else None
        rgb, feat = mrs.render(gs, W, H, spp, 3, 9, want_aux=aux, out_sumsq=sq, out_layers=lay,
                               accum_fp64=fp64)
        torch.cuda.synchronize()
        return [t for t in (rgb, sq, feat, lay) if t is not None]

    try:
        one = outputs(streams=1)
        assert all(torch.isfinite(t).all() for t in one) and float(one[0].sum()) > 0
        inside = 0
        for tuning in (dict(streams=2), dict(streams=3), dict(streams=4),
                       dict(streams=3, chunk_paths=300_000)):
            k, chunk = tuning["streams"], tuning.get("chunk_paths", total)
            sub = -(-min(chunk, total) // k) + 255 & ~255  # paths of a sub-chunk
            assert total > 1 << 18 and total // 65536 >= k  # this many streams
            inside += any(c % spp for c in range(sub, total, sub))
            got = outputs(**tuning)
            assert all(torch.equal(a, b) for a, b in zip(got, one)), tuning
        assert inside >= 3  # of the four cut a pixel
    finally:
        mrs.set_tuning(**old)
