"""A layer's data gradient, weight gradient and the earlier layer's sum in one launch
(k_layer_bwd) against the separate kernels (which larger tiles run on): bitwise the same
gradients, on a first and on a repeated pass."""
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


# LR sizes: rows of 8 pixels (the fast weight gradient), of other lengths (separate
# kernels throughout), one split and several, more pixels than a split holds
@pytest.mark.parametrize("arch", ["res16", "rdg_x2", "res16_layers"])
@pytest.mark.parametrize("B,h,w", [(1, 1, 8), (3, 5, 8), (1, 9, 24), (2, 8, 12), (2, 40, 32)])
def test_one_launch_matches_separate_kernels(mrs, arch, B, h, w):
    import torch
    net = mrs.FusionNet(seed=4, arch=arch)
    s = net.scale
    g = torch.Generator(device="cuda").manual_seed(7 * h + w)
    r = lambda *shape: torch.rand(*shape, generator=g, device="cuda")
    H, W = h * s, w * s
    x = (r(B, H, W, 3), r(B, H, W, 7), r(B, h, w, 3), r(B, H, W, 3))
    lay = (r(B, H, W, 9), r(B, H, W, 3), 4) if net.has_layers else None
    got = []
    for tiles in (1 << 30, 0, 1 << 30):
        mrs.set_tuning(conv_small_tiles=tiles, net_fused_blocks=0)
        grad, loss, _ = net.loss_grad(*x, layers=lay)
        assert np.isfinite(grad).all() and np.abs(grad).max() > 0
        got.append((grad, loss))
    for grad, loss in got[1:]:
        assert np.array_equal(grad, got[0][0]) and loss == got[0][1]
