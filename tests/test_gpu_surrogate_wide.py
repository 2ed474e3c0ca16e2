"""The convolution kernel for layers with many pixels (256-pixel tiles,
workgroups running through several tiles) against the direct kernel on the
same network: tiles of 8 x 32 and 16 x 16, image and tile edges with both
paddings, counts of work items that do not divide by the workgroups."""
import numpy as np
import pytest

from paper_2408_01081_amd import surrogate as S

gpu = pytest.mark.gpu


def _torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _net(B, H, W, split, mode, train=False):
    P = S.init_params(seed=3, out_scale=0.3)
    g = np.random.default_rng(4)
    for k in P:
        if k.endswith(".a"):
            P[k] = P[k] + 0.1 * g.standard_normal(P[k].shape)
    net = S.Surrogate(B, H, W, split=split, train=train)
    net.set_params(S.pack_params(P))
    return net.set_conv_mode(mode)


def _input(torch, B, H, W, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.randn(B, 8, H, W, device="cuda", generator=g)
    x[:, 5] = torch.rand(B, 1, 1, device="cuda", generator=g) + 0.1
    x[:, 6], x[:, 7] = 1.0, 1.5
    return x


# Both kernels form the same products (hi/lo splits of the same FP32 values)
# and differ in the order of FP32 sums of up to n = 27 * 128 terms: about
# sqrt(n) / 2 roundings of 2^-24 per layer, 2e-6, over 16 layers 8e-6 in the
# mean; a layer's differing output may also round to another lo part (2^-17
# of it, in few values).
TOL = 3e-5


@gpu
@pytest.mark.parametrize("B,H,W,circular", [(1, 256, 256, True), (1, 256, 256, False),
                                            (9, 128, 128, False), (21, 64, 384, True),
                                            (33, 64, 128, False)])
def test_wide_convolution_matches_direct(B, H, W, circular):
    torch = _torch()
    x = _input(torch, B, H, W, B + W)
    outs = [_net(B, H, W, 3, mode).forward(x, circular=circular) - x[:, :5] for mode in (0, 1)]
    err = float((outs[0].double() - outs[1].double()).norm() / outs[1].double().norm())
    print("B %d %dx%d: %.2e" % (B, H, W, err))
    assert err < TOL


@gpu
def test_wide_convolution_plain_bf16_matches_reference():
    # plain BF16 operands: each layer's rounding decisions depend on the order
    # of the sums before it, so the comparison is with the FP64 reference, at
    # the tolerance of the forward test for such operands (tests/test_gpu_surrogate.py)
    torch = _torch()
    from oracle import surrogate_ref as R
    B, H, W = 5, 128, 128
    x = _input(torch, B, H, W, 7)
    net = _net(B, H, W, 1, 0)
    out = (net.forward(x) - x[:, :5]).double().cpu().numpy()
    P = {k: v.astype(np.float64) for k, v in S.unpack_params(net.get_params().cpu().numpy()).items()}
    xin = x.double().cpu().numpy()
    ref = R.Forward(P, xin, True).out - xin[:, :5]
    assert np.linalg.norm(out - ref) < 3e-2 * np.linalg.norm(ref)


@gpu
@pytest.mark.parametrize("circular", [True, False])
def test_wide_gradients_match_direct(circular):
    torch = _torch()
    B, H, W = 9, 128, 128
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
        # the backward pass adds its own 16 layers: twice the sums
        assert err < 2 * TOL, (k, err)


@gpu
def test_gradients_match_reference_odd_batch():
    # FiLM sums of a batch that is no multiple of the 8 samples a workgroup
    # takes at a time, against the FP64 reference at the tolerance of the
    # gradient test (tests/test_gpu_surrogate.py)
    torch = _torch()
    from oracle import surrogate_ref as R
    B, H, W = 9, 64, 128
    x = _input(torch, B, H, W, 5)
    g = torch.Generator(device="cuda").manual_seed(6)
    t = x[:, :5] + 0.1 * torch.randn(B, 5, H, W, device="cuda", generator=g)
    net = _net(B, H, W, 3, 0, train=True)
    P = {k: v.astype(np.float64) for k, v in S.unpack_params(net.get_params().cpu().numpy()).items()}
    net.train_step(x, t, circular=False, lr=0.0)
    G = S.unpack_params(net.get_grads().double().cpu().numpy())
    ref = R.Forward(P, x.double().cpu().numpy(), False)
    ref.loss(t.double().cpu().numpy())
    want = ref.backward()
    for k in want:
        n = np.linalg.norm(want[k])
        assert np.linalg.norm(G[k] - want[k]) <= 1e-3 * n, k
