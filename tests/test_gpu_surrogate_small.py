"""The convolution kernel for layers with few pixels (all input chunks at once,
4 or 8 rows x 16 pixels per workgroup) against the direct kernel on the same
network: from the smallest image, whose every layer takes it, to a batch whose
coarsest layers do; the statistics of images of 32 to more than 256 chunks."""
import numpy as np
import pytest

from paper_2408_01081_amd import surrogate as S
from test_gpu_surrogate_wide import TOL, _input, _net, _torch

gpu = pytest.mark.gpu


# tolerance: the same products as the direct kernel's, another order of sums
# (see TOL)
@gpu
@pytest.mark.parametrize("B,H,W,circular", [(1, 64, 128, True), (1, 64, 128, False),
                                            (2, 192, 128, False), (3, 64, 256, True),
                                            (34, 64, 128, True), (1, 320, 256, False)])
def test_small_convolution_matches_direct(B, H, W, circular):
    torch = _torch()
    x = _input(torch, B, H, W, B + H)
    outs = [_net(B, H, W, 3, mode).forward(x, circular=circular) - x[:, :5] for mode in (0, 1)]
    err = float((outs[0].double() - outs[1].double()).norm() / outs[1].double().norm())
    print("B %d %dx%d: %.2e" % (B, H, W, err))
    assert err < TOL


@gpu
@pytest.mark.parametrize("B,H,W,circular", [(1, 64, 128, True), (2, 192, 128, False),
                                            (34, 64, 128, False)])
def test_small_gradients_match_direct(B, H, W, circular):
    torch = _torch()
    x = _input(torch, B, H, W, 1)
    g = torch.Generator(device="cuda").manual_seed(2)
    t = x[:, :5] + 0.1 * torch.randn(B, 5, H, W, device="cuda", generator=g)
    grads = []
    for mode in (0, 1):
        net = _net(B, H, W, 3, mode, train=True)
        net.train_step(x, t, circular=circular, lr=0.0)
        grads.append(S.unpack_params(net.get_grads().double().cpu().numpy()))
    for k in grads[0]:
        n = np.linalg.norm(grads[1][k])
        err = np.linalg.norm(grads[0][k] - grads[1][k]) / max(n, 1e-30)
        assert err < 2 * TOL, (k, err)


@gpu
@pytest.mark.parametrize("H,W", [(512, 512), (512, 640)])
def test_gain_gradients_of_large_images_match_direct(H, W):
    # up to 1024 tiles per sample the convolution forms the gain gradient's
    # chunk sums, beyond that a kernel of their own
    torch = _torch()
    x = _input(torch, 1, H, W, 3)
    g = torch.Generator(device="cuda").manual_seed(4)
    t = x[:, :5] + 0.1 * torch.randn(1, 5, H, W, device="cuda", generator=g)
    grads = []
    for mode in (0, 1):
        net = _net(1, H, W, 3, mode, train=True)
        net.train_step(x, t, circular=False, lr=0.0)
        grads.append(S.unpack_params(net.get_grads().double().cpu().numpy()))
    for k in grads[0]:
        n = np.linalg.norm(grads[1][k])
        err = np.linalg.norm(grads[0][k] - grads[1][k]) / max(n, 1e-30)
        assert err < 2 * TOL, (k, err)


@gpu
@pytest.mark.parametrize("B,H,W,circular", [(1, 256, 256, False), (5, 384, 128, True),
                                            (33, 64, 128, False), (2, 64, 128, True)])
def test_plain_bf16_sums_keep_their_order(B, H, W, circular):
    # with plain BF16 operands the order of a layer's sums decides the
    # roundings of all layers after it: the wide kernel adds its products as
    # the 64-pixel kernel does (mode 2), and the fused epilogues do what their
    # kernels did, so the two give the same bits
    torch = _torch()
    x = _input(torch, B, H, W, B)
    outs = [_net(B, H, W, 1, mode).forward(x, circular=circular) for mode in (0, 2)]
    assert torch.equal(outs[0], outs[1])
