"""Per-pixel sums: the kernel with a thread per pixel and the one with 16 lanes per pixel
add the same samples in the same order, whether the sums go straight to the outputs (all
paths resident) or through memory (several super-chunks), so every output is bitwise
the same."""
import pytest

from mrs_inputs import scenes as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.mark.parametrize("spp", [1, 15, 16, 17, 31, 32, 33, 49])
@pytest.mark.parametrize("fp64", [0, 1])
def test_sums_are_bitwise_the_same_on_every_route(torch_cuda, spp, fp64):
    """37 x 21 pixels (ragged tiles, a last block that is not full).  From 16 to 31
    samples the radiance alone takes the thread-per-pixel kernel and the render with
    features and layers the 16-lane one."""
    import paper_2106_12802_amd as mrs
    torch = torch_cuda
    gs = mrs.GpuScene(S.procedural(7, spheres=((2, 3),), n_boxes=4, n_lights=2))
    W, H, D, seed = 37, 21, 4, 100 + spp

    def outputs(aux, layers):
        sq = torch.full((H, W, 3), float("nan"), device="cuda")
        lay = torch.full((H, W, 9), float("nan"), device="cuda") if layers else None
        rgb, feat = mrs.render(gs, W, H, spp, D, seed, want_aux=aux, out_sumsq=sq,
                               out_layers=lay, accum_fp64=fp64)
        torch.cuda.synchronize()
        return [rgb, sq] + ([feat] if aux else []) + ([lay] if layers else [])

    full = outputs(True, True)
    assert all(torch.isfinite(t).all() for t in full) and float(full[3].abs().sum()) > 0
    routes = [outputs(False, False), outputs(True, False), outputs(False, True)]
    old = mrs.get_tuning()
    try:
        # super-chunks of several pixels, of less than a pixel's samples, and three
        # sub-chunks a super-chunk (cut inside pixels)
        for chunk in (1000, 256, W * H * spp // 2 + 3):
            mrs.set_tuning(chunk_paths=chunk)
            again = outputs(True, True)
            assert all(torch.equal(a, b) for a, b in zip(full, again)), chunk
            routes.append(outputs(False, False))
    finally:
        mrs.set_tuning(**old)
    for r in routes:
        assert torch.equal(r[0], full[0]) and torch.equal(r[1], full[1])
    assert torch.equal(routes[1][2], full[2]) and torch.equal(routes[2][2], full[3])


@pytest.mark.parametrize("spp", [7, 40])
def test_sums_of_pixels_cut_by_concurrent_sub_chunks(torch_cuda, spp):
    """Enough paths for three concurrent sub-chunks whose ends fall inside pixels."""
    import paper_2106_12802_amd as mrs
    torch = torch_cuda
    gs = mrs.GpuScene(S.cornell(2))
    n = 200_000 // spp
    H = 101
    W = n // H
    old = mrs.get_tuning()
    try:
        mrs.set_tuning(streams=3)
        three = mrs.render(gs, W, H, spp, 3, 9)
        torch.cuda.synchronize()
        mrs.set_tuning(streams=1)
        one = mrs.render(gs, W, H, spp, 3, 9)
        torch.cuda.synchronize()
    finally:
        mrs.set_tuning(**old)
    assert torch.equal(three[0], one[0]) and torch.equal(three[1], one[1])


def test_sums_of_mixed_jobs(torch_cuda):
    """A batch whose jobs take different sum kernels in turn equals its single renders."""
    import paper_2106_12802_amd as mrs
    torch = torch_cuda
    gs = mrs.GpuScene(S.cornell(1))
    jobs = [dict(scene=gs, W=33, H=9, spp=s, max_depth=3, seed=50 + i)
            for i, s in enumerate((4, 40, 3, 1030, 20, 2))]
    b = mrs.Batch(jobs)
    for _ in range(2):
        b.render()
    torch.cuda.synchronize()
    for j, (rgb, aux) in zip(jobs, b.outputs):
        r1, a1 = mrs.render(gs, j["W"], j["H"], j["spp"], 3, j["seed"])
        torch.cuda.synchronize()
        assert torch.equal(rgb, r1) and torch.equal(aux, a1)
