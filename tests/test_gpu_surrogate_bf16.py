"""A training step with plain BF16 operands: gradients against the FP64 reference
and against the direct kernels on the same activations, over both tile widths of
the weight-gradient kernel (32 x 8 and 16 x 16 pixels), odd batches and both
paddings."""
import numpy as np
import pytest

from paper_2408_01081_amd import surrogate as S

gpu = pytest.mark.gpu


def _torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _step(torch, B, H, W, circular, mode):
    P = S.init_params(seed=3, out_scale=0.3)
    g = np.random.default_rng(4)
    for k in P:
        if k.endswith(".a"):
            P[k] = P[k] + 0.1 * g.standard_normal(P[k].shape)
    net = S.Surrogate(B, H, W, split=1, train=True)
    net.set_params(S.pack_params(P))
    net.set_conv_mode(mode)
    gen = torch.Generator(device="cuda").manual_seed(B + W)
    x = torch.randn(B, 8, H, W, device="cuda", generator=gen)
    x[:, 5] = torch.rand(B, 1, 1, device="cuda", generator=gen) + 0.1
    x[:, 6], x[:, 7] = 1.0, 1.5
    t = x[:, :5] + 0.1 * torch.randn(B, 5, H, W, device="cuda", generator=gen)
    net.train_step(x, t, circular=circular, lr=0.0)
    params = S.unpack_params(net.get_params().cpu().numpy())
    return x, t, params, S.unpack_params(net.get_grads().double().cpu().numpy())


# The forward test's tolerance for such operands is 3e-2 over 16 layers; the
# gradients pass through 16 more.
@gpu
@pytest.mark.parametrize("B,H,W,circular", [(9, 128, 128, True), (3, 64, 256, False)])
def test_plain_bf16_gradients_match_reference(B, H, W, circular):
    torch = _torch()
    from oracle import surrogate_ref as R
    x, t, params, G = _step(torch, B, H, W, circular, 0)
    P = {k: v.astype(np.float64) for k, v in params.items()}
    ref = R.Forward(P, x.double().cpu().numpy(), circular)
    ref.loss(t.double().cpu().numpy())
    want = ref.backward()
    for k in want:
        n = np.linalg.norm(want[k])
        err = np.linalg.norm(G[k] - want[k])
        print(k, err / n)
        assert err <= 6e-2 * n, k


# With so many pixels the direct kernel slices no layer's reduction (it needs 1024
# workgroups of 128 pixels x 16 channels at every level, 2^20 pixels in all), and
# the tiled kernels add a layer's products in its order, so both modes have the
# same activations and the same dL/dy, bit for bit; a weight's sum of n = B H W FP32
# products differs by its order, sqrt(n) / 2 roundings of 2^-24 in the mean, of
# which four times are allowed.
@gpu
@pytest.mark.parametrize("B,H,W,circular", [(65, 128, 128, True), (65, 128, 128, False),
                                            (33, 128, 256, False)])
def test_plain_bf16_weight_gradients_match_direct(B, H, W, circular):
    torch = _torch()
    got, want = (_step(torch, B, H, W, circular, mode)[3] for mode in (0, 1))
    for k in want:
        n = np.linalg.norm(want[k])
        err = np.linalg.norm(got[k] - want[k])
        print(k, err / n)
        assert err <= 2 * np.sqrt(B * H * W) * 2.0 ** -24 * n, k
