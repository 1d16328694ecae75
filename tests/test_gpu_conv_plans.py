"""The 3x3 convs of 64-channel slices (k_conv3_rw): their tile plans sum every
output in one K order, forward and backward, so results are bitwise alike; images
too wide for a tile's 31-bit offsets run on the direct convs."""
import numpy as np
import pytest

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


def _inputs(seed, B, H, W, s):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    r = lambda *shape: torch.rand(*shape, generator=g, device="cuda")
    return r(B, H, W, 3), r(B, H, W, 7), r(B, H // s, W // s, 3), r(B, H, W, 3)


# LR sizes at the edges of the 16 x 16 and 16 x 8 tiles: one pixel, one short of a
# tile, one tile, one over, several images
@pytest.mark.parametrize("arch", ["res16", "rdg", "rdg_x2"])
@pytest.mark.parametrize("B,h,w", [(1, 1, 1), (2, 7, 15), (1, 16, 16), (3, 9, 17), (1, 33, 31)])
def test_plans_agree_bitwise(mrs, arch, B, h, w):
    import torch
    net = mrs.FusionNet(seed=5, arch=arch)
    s = net.scale
    x = _inputs(11 * h + w, B, h * s, w * s, s)
    got = []
    for tiles in (0, 1 << 30):
        mrs.set_tuning(conv_small_tiles=tiles, net_fused_blocks=0)
        mrs.tracer.conv_launches(reset=True)
        grad, loss, out = net.loss_grad(*x)
        ran = mrs.tracer.conv_launches(reset=True)
        used, other = ("large", "small") if tiles == 0 else ("small", "large")
        assert ran[f"lds64_{used}"] > 30 and ran[f"dgrad_lds_{used}"] > 30, ran
        assert ran[f"lds64_{other}"] == 0 and ran[f"dgrad_lds_{other}"] == 0, ran
        assert np.isfinite(grad).all() and np.isfinite(loss)
        got.append((grad, loss, out.clone()))
    assert np.array_equal(got[0][0], got[1][0]) and got[0][1] == got[1][1]
    assert torch.equal(got[0][2], got[1][2])


def test_wide_images_run_on_the_direct_convs(mrs):
    """2^31 bytes / (18 rows x 256 channels x 4 bytes) = 116,508 pixels.  The direct
    conv sums its channels in another order: two BF16 evaluations of one network,
    each within 5e-3 of the exact one and mostly rounded alike (bar 2e-3)."""
    import torch
    net = mrs.FusionNet(seed=5, arch="rdg_x2")
    w, crop, margin = 116_512, 1024, 160  # the network sees about 70 LR pixels
    x = _inputs(3, 1, 2, 2 * w, 2)
    mrs.tracer.conv_launches(reset=True)
    grad, loss, out = net.loss_grad(*x)
    ran = mrs.tracer.conv_launches(reset=True)
    assert ran["lds64_large"] == ran["lds64_small"] == 0 and ran["direct64"] > 60, ran
    assert np.isfinite(grad).all()
    cut = [t[:, :, :t.shape[2] // w * crop].contiguous() for t in x]
    _, _, ref = net.loss_grad(*cut)
    a, b = out[:, :, :2 * (crop - margin)], ref[:, :, :2 * (crop - margin)]
    err = float((a - b).norm() / b.norm())
    assert err <= 2e-3, err


# HR / LR sizes at the edges of the 32 x 16 input tiles, the 16 x 16 reconstruction
# tiles and the fuse conv's 128-pixel blocks: one LR pixel, one short of a tile, one
# over, several images
@pytest.mark.parametrize("arch,B,h,w", [
    ("res16", 1, 1, 1), ("res16", 2, 3, 9), ("res16", 1, 17, 8), ("res16", 3, 9, 5),
    ("rdg", 1, 1, 1), ("rdg", 2, 5, 13), ("rdg_x2", 1, 1, 2), ("rdg_x2", 2, 17, 9),
    ("rdg_x8", 1, 1, 1), ("rdg_x8", 2, 3, 5)])
def test_input_fuse_and_reconstruction_edges(mrs, arch, B, h, w):
    """Against the oracle.  The BF16 network is within 5e-3 (16 blocks) and 8e-3
    (dense groups) of it over whole images; a few LR pixels average over as few as
    12 values, so the bar here is four times that of the latter.  A misplaced
    channel or pixel is off by order one."""
    import torch
    from oracle import cnn, cnn_rdg
    net = mrs.FusionNet(seed=9, arch=arch)
    s = net.scale
    x = _inputs(17 * h + w, B, h * s, w * s, s)
    out = net.fuse(*x[:3]).cpu().numpy().astype(np.float64)
    torch.cuda.synchronize()
    hr, aux, lr = (t.cpu().numpy() for t in x[:3])
    params = net.get_params().astype(np.float64)
    ref = (cnn.forward(params, hr, aux, lr) if arch == "res16"
           else cnn_rdg.forward(params, hr, aux, lr, scale=s))
    ref = ref[0] if isinstance(ref, tuple) else ref
    err = np.linalg.norm(out - ref) / np.linalg.norm(ref)
    assert err <= 3.2e-2, err
