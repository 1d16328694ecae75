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


@pytest.mark.parametrize("arch", ["res16", "rdg_x2"])
def test_direct_data_gradients_of_wide_images(mrs, arch):
    """Images wider than 116,508 pixels run the direct data-gradient kernel in every layer.
    An output gradient that is zero outside a window gives the parameter gradient of a
    crop around it.  The two sum in another order, which flips about one BF16 rounding
    in 1e4 (4e-3 each) in each of ~100 tensors: 4e-4 of the norm; the bar is 2e-3."""
    import torch
    net = mrs.FusionNet(seed=6, arch=arch)
    s, h, w, crop, margin = net.scale, 2, 116_512, 512, 160
    g = torch.Generator(device="cuda").manual_seed(3)
    r = lambda *shape: torch.rand(*shape, generator=g, device="cuda")
    x = [r(1, h * s, w * s, 3), r(1, h * s, w * s, 7), r(1, h, w, 3)]
    go = torch.zeros(1, h * s, w * s, 3, device="cuda")
    go[:, :, :s * (crop - margin)] = r(1, h * s, s * (crop - margin), 3) - 0.3
    mrs.tracer.conv_launches(reset=True)
    wide = net.backward(*x, go)
    ran = mrs.tracer.conv_launches(reset=True)
    assert ran["dgrad_lds_small"] == ran["dgrad_lds_large"] == 0, ran
    cut = [t[:, :, :t.shape[2] // w * crop].contiguous() for t in x]
    ref = net.backward(*cut, go[:, :, :s * crop].contiguous())
    err = float(np.linalg.norm(wide - ref) / np.linalg.norm(ref))
    assert err <= 2e-3, err


@pytest.mark.parametrize("arch", ["res16", "rdg", "rdg_x2", "rdg_x8"])
@pytest.mark.parametrize("h,w", [(3, 8), (5, 12)])
def test_weight_gradient_views(mrs, arch, h, w):
    """LR rows of a multiple of 8 pixels (views by shifts in every layer) and not (the LR
    layers by view_ptr): a batch's gradient is the sum of its images' (FP32 sums in
    another order, ~1e-7 of the norm each; a pixel of the wrong image or place is off by
    order one; bar 1e-5)."""
    import torch
    net = mrs.FusionNet(seed=8, arch=arch)
    s = net.scale
    g = torch.Generator(device="cuda").manual_seed(h + w)
    r = lambda *shape: torch.rand(*shape, generator=g, device="cuda")
    H, W = h * s, w * s
    x = (r(2, H, W, 3), r(2, H, W, 7), r(2, h, w, 3))
    go = r(2, H, W, 3) - 0.5
    both = net.backward(*x, go)
    one = [net.backward(*(t[i:i + 1].contiguous() for t in x), go[i:i + 1].contiguous())
           for i in range(2)]
    want = one[0].astype(np.float64) + one[1]
    assert np.linalg.norm(both - want) <= 1e-5 * np.linalg.norm(want)
