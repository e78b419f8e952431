"""The bf16 weight gradient where a workgroup goes down an image and finds two rows of the aggregates from the strip above: images of several
strips with a short last one, slices that begin and end inside an image, both numbers of input-channel blocks, with and without the max pool.
beta = 1/2, so that the aggregates are exact in bf16; against sums in 64 bits over the dL/dY that the call returned, rounded as the kernel does."""
import pytest
import torch

from paper_2603_13810_amd import api

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
BITS, MAX = api.TAC_IN_BITS, api.TAC_IN_BITS_MAXPOOL2

# (B, Cin, Cout, H, W, format, K, T)
CASES = [
    (4, 32, 256, 40, 16, BITS, 4, 8),
    (3, 32, 128, 45, 32, BITS, 4, 9),
    (3, 64, 128, 45, 32, MAX, 2, 7),
    (5, 64, 128, 37, 64, BITS, 4, 14),
    (2, 32, 128, 66, 64, MAX, 3, 5),
    (2, 96, 128, 21, 128, BITS, 7, 9),
    (2, 32, 128, 23, 128, MAX, 3, 5),
    (65, 64, 128, 125, 32, MAX, 2, 4),        # 2048 strips and more: two blocks of input channels
    (43, 64, 128, 93, 64, BITS, 4, 8),
]


@pytest.mark.parametrize("case", CASES, ids=["%d_to_%d_%dx%d_f%d" % c[1:6] for c in CASES])
def test_weight_gradient_over_strips(case):
    B, Cin, Cout, H, W, fmt, K, T = case
    r = torch.Generator(device=DEV)
    r.manual_seed(7900 + Cin + Cout + H + W)
    f = 2 if fmt == MAX else 1
    x = [(torch.rand((B, Cin, f * H, f * W), generator=r, device=DEV) < 0.2).to(torch.uint8) for _ in range(T)]
    desc = api.make_desc(T, B, Cin, H, W, Cout, K=K, beta=0.5, theta=1.0, mode=api.TAC_COLLAPSE, in_format=fmt, precision=api.TAC_BF16)
    G = api.tac_out_shape(desc)[0]
    v = 0.6 * torch.randn((G, B, Cout, H, W), generator=r, device=DEV) + 0.3
    g = torch.randn(v.shape, generator=r, device=DEV)
    w = 0.1 * torch.randn((Cout, Cin, 3, 3), generator=r, device=DEV)
    got = api.tac_conv_lif_backward(desc, torch.stack([api.tac_pack_spikes(a) for a in x]), w, v, g, want_input_grad=False)
    dW = torch.zeros((Cout, Cin, 9), dtype=torch.float64, device=DEV)
    dabs = torch.zeros_like(dW)
    for k in range(G):
        frames = x[k * K:(k + 1) * K]
        if fmt == MAX:
            frames = [torch.nn.functional.max_pool2d(a.float(), 2) for a in frames]
        A = torch.zeros((B, Cin, H + 2, W + 2), dtype=torch.float64, device=DEV)
        A[:, :, 1:-1, 1:-1] = sum(0.5 ** (len(frames) - 1 - j) * a.double() for j, a in enumerate(frames))
        dY = got["grad_y"][k].bfloat16().double().transpose(0, 1).reshape(Cout, -1)
        for t in range(9):
            a = A[:, :, t // 3:t // 3 + H, t % 3:t % 3 + W].transpose(0, 1).reshape(Cin, -1).t().contiguous()
            dW[:, :, t] += dY @ a
            dabs[:, :, t] += dY.abs() @ a
    # sums of n fp32 terms in any order: 2^-24 sqrt(n) of the sum of the magnitudes, times four
    tol = 4 * 2.0 ** -24 * (G * B * H * W) ** 0.5
    err = (got["grad_w"].double().flatten(2) - dW).abs()
    assert (err <= tol * dabs + 1e-12).all(), float((err / dabs).max() / tol)
