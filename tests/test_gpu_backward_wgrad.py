"""The fp32 matrix-core weight gradient at the edges of its tiles: one column tile and many, channel counts that fill no
tile, strips and row segments with a remainder, both strides, every way to load, shorter last groups; against the
gradient that automatic differentiation of a double-precision convolution gives for the same dL/dY."""
import numpy as np
import pytest
import torch

from paper_2603_13810_amd import api
from parity_util import np_pack

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
BITS, MEAN, MAX, REAL = api.TAC_IN_BITS, api.TAC_IN_BITS_POOL2, api.TAC_IN_BITS_MAXPOOL2, api.TAC_IN_F32

# (B, Cin, Cout, H, W, stride, format, K, T)
CASES = [
    (3, 1, 5, 9, 11, 1, BITS, 2, 5),          # one column tile, eight waves over the pixels
    (2, 3, 40, 30, 70, 1, BITS, 4, 6),        # two row segments
    (2, 2, 70, 13, 21, 2, REAL, 3, 7),
    (2, 4, 33, 7, 14, 1, REAL, 2, 4),         # two tiles
    (2, 8, 24, 10, 31, 2, MEAN, 4, 4),        # three tiles, one channel block
    (1, 24, 64, 6, 132, 1, MAX, 1, 3),        # three segments, two channel blocks
    (2, 37, 130, 5, 5, 1, BITS, 8, 11),       # column groups that start inside a channel, a channel block of two
    (1, 72, 96, 3, 2, 1, BITS, 16, 17),
    (2, 32, 64, 14, 14, 1, MEAN, 4, 7),
    (1, 512, 512, 2, 2, 1, BITS, 2, 4),       # few neurons: dW is cleared by a launch of its own
]


@pytest.mark.parametrize("case", CASES, ids=["%d_to_%d_%dx%d_s%d_f%d" % c[1:7] for c in CASES])
def test_weight_and_bias_gradient(case):
    B, Cin, Cout, H, W, stride, fmt, K, T = case
    r = np.random.Generator(np.random.PCG64(7000 + Cin + Cout + H + W))
    f = 2 if fmt in (MEAN, MAX) else 1
    x = (r.random((T, B, Cin, f * H, f * W)) < 0.3).astype(np.float32)
    if fmt == REAL:
        x *= r.random(x.shape).astype(np.float32)
    xd = torch.from_numpy(x if fmt == REAL else np_pack(x.astype(np.uint8))).to(DEV)
    desc = api.make_desc(T, B, Cin, H, W, Cout, K=K, beta=0.9, theta=1.0, mode=api.TAC_COLLAPSE, stride=stride, in_format=fmt)
    T_out, Ho, Wo = api.tac_out_shape(desc)
    v = (0.6 * r.standard_normal((T_out, B, Cout, Ho, Wo)) + 0.3).astype(np.float32)
    g = r.standard_normal(v.shape).astype(np.float32)
    w = (r.standard_normal((Cout, Cin, 3, 3)) * 0.1).astype(np.float32)
    stale = torch.full((Cout, Cin, 3, 3), float("nan"), device=DEV)       # what the allocator hands out next
    del stale
    got = api.tac_conv_lif_backward(desc, xd, torch.from_numpy(w).to(DEV), torch.from_numpy(v).to(DEV), torch.from_numpy(g).to(DEV),
                                    want_input_grad=False)
    torch.cuda.synchronize()
    gy = got["grad_y"].cpu().double()
    frames = torch.from_numpy(x).double()
    if fmt == MEAN:
        frames = torch.nn.functional.avg_pool2d(frames.flatten(0, 2)[:, None], 2).view(T, B, Cin, H, W)
    if fmt == MAX:
        frames = torch.nn.functional.max_pool2d(frames.flatten(0, 2)[:, None], 2).view(T, B, Cin, H, W)
    beta = float(np.float32(0.9))
    dW = torch.zeros((Cout, Cin, 3, 3), dtype=torch.float64)
    dabs = torch.zeros_like(dW)
    for k in range(T_out):
        Kg = min(K, T - k * K)
        A = sum(beta ** (Kg - 1 - j) * frames[k * K + j] for j in range(Kg))
        for dst, a, b in ((dW, A, gy[k]), (dabs, A.abs(), gy[k].abs())):
            wv = torch.zeros((Cout, Cin, 3, 3), dtype=torch.float64, requires_grad=True)
            torch.nn.functional.conv2d(a, wv, None, stride, 1).backward(b)
            dst += wv.grad
    # sums of n fp32 terms in any order, each term and aggregate rounded a few times: 2^-24 (sqrt(n) + K) of the sum of
    # the magnitudes, times four
    n = T_out * B * Ho * Wo
    tol = 4 * 2.0 ** -24 * (n ** 0.5 + K)
    assert ((got["grad_w"].cpu().double() - dW).abs() <= tol * dabs + 1e-12).all()
    db, dbabs = gy.sum((0, 1, 3, 4)), gy.abs().sum((0, 1, 3, 4))
    assert ((got["grad_bias"].cpu().double() - db).abs() <= tol * dbabs).all()


def test_an_infinite_frame_value_stays_where_it_is():
    # 5 pixels a row: the pixels that fill the row's last quad must not multiply the infinite value by zero
    B, Cin, Cout, H, W = 1, 2, 8, 5, 5
    x = torch.rand((1, B, Cin, H, W), device=DEV)
    x[0, 0, 1, 2, 4] = float("inf")
    desc = api.make_desc(1, B, Cin, H, W, Cout, K=1, beta=0.9, theta=1.0, mode=api.TAC_PER_STEP, in_format=REAL)
    v = torch.zeros((1, B, Cout, H, W), device=DEV)
    got = api.tac_conv_lif_backward(desc, x, torch.zeros((Cout, Cin, 3, 3), device=DEV), v, torch.ones_like(v), want_input_grad=False)
    gw = got["grad_w"].cpu()
    assert torch.isfinite(gw[:, 0]).all()
    # column kx = 0 sees input pixels 0 .. 3 of a row (x = 1 .. 4), never the last one
    assert torch.isfinite(gw[:, 1, :, 0]).all() and torch.isinf(gw[:, 1, :, 1:]).all()


@pytest.mark.parametrize("B,Cin,Cout,hw,T,rate", [(16, 256, 256, 40, 4, 0.12), (100, 256, 128, 32, 2, 1.0),
                                                    # first layers, 640 and 520 products a thread
                                                    (640, 1, 128, 64, 2, 1.0), (520, 2, 64, 64, 4, 0.12)])
def test_long_sums_of_one_sign(B, Cin, Cout, hw, T, rate):
    # 1e5 pixels and more per element, all terms positive: a sum that is one long chain of additions loses digits here.
    # dL/dY is the same everywhere within a step, so that dW is that value times the number of spikes under the tap.
    r = np.random.Generator(np.random.PCG64(7100 + hw))
    x = (r.random((T, B, Cin, hw, hw)) < rate).astype(np.uint8)
    desc = api.make_desc(T, B, Cin, hw, hw, Cout, K=1, beta=0.9, theta=1.0, mode=api.TAC_PER_STEP)
    v = torch.full((T, B, Cout, hw, hw), 0.4, device=DEV)
    got = api.tac_conv_lif_backward(desc, torch.from_numpy(np_pack(x)).to(DEV), torch.zeros((Cout, Cin, 3, 3), device=DEV), v,
                                    torch.full_like(v, 0.37), want_input_grad=False, detach_reset=True)
    gy = got["grad_y"].flatten(1)
    assert (gy > 0).all() and torch.equal(gy, gy[:, :1].expand_as(gy))
    per_step = gy[:, 0].double().cpu().numpy()
    padded = np.pad(x, ((0, 0), (0, 0), (0, 0), (1, 1), (1, 1)))
    count = np.stack([padded[:, :, :, ky:ky + hw, kx:kx + hw].sum((1, 3, 4), dtype=np.int64) for ky in range(3) for kx in range(3)], -1)
    dW = np.broadcast_to((per_step[:, None, None] * count).sum(0), (Cout, Cin, 9))
    db = per_step.sum() * B * hw * hw
    # Chains of at most some 64 MFMAs (first layers: products, whose sums meet in 64 bits), 64 sums of chains, 8 waves and 48 slices (first layers: 64) follow one
    # another; n additions, each
    # rounded by up to 2^-24 of the sum so far, leave about 2^-24 sqrt(n) of it: n < 256
    tol = 16 * 2.0 ** -24
    err = got["grad_w"].double().cpu().numpy().reshape(dW.shape) - dW
    assert np.linalg.norm(err) <= tol * np.linalg.norm(dW)
    assert np.abs(got["grad_bias"].double().cpu().numpy() - db).max() <= tol * db


# first layers: quads with a remainder and at odd addresses, one and several groups of channels, strips, several pairs per item, a
# shorter last group, both strides, bits and real values (those of 2 -> 96 stride 2 and 2 -> 300 outweigh dL/dY: the other kernel's)
FIRST = [
    (3, 1, 5, 9, 11, 1, BITS, 2, 5), (5, 1, 33, 28, 28, 1, BITS, 4, 9), (2, 2, 130, 13, 70, 1, BITS, 3, 7), (1, 2, 16, 100, 100, 2, BITS, 8, 9),
    (2, 2, 64, 33, 31, 1, REAL, 2, 5), (1, 1, 128, 64, 64, 1, REAL, 4, 6), (3, 2, 96, 7, 9, 2, REAL, 1, 3), (70, 1, 8, 5, 4, 1, BITS, 1, 2),
    (1, 1, 4, 1, 1, 1, BITS, 1, 1), (2, 2, 300, 6, 12, 1, REAL, 16, 17),
    # real-valued frames on 128 workgroups and more
    (24, 2, 64, 33, 31, 1, REAL, 2, 5), (40, 1, 128, 40, 24, 2, REAL, 4, 6), (60, 2, 96, 7, 9, 1, REAL, 1, 3),
    # bits of two input channels on 64 workgroups and more (those of 2 -> 16 stride 2 are fewer)
    (16, 2, 52, 51, 57, 2, BITS, 16, 17),
]

# which of them run on the first layers' kernel (the choice is held to this on the CPU)
FIRST_TAKEN = [True, True, True, False, False, False, False, True, True, False, True, True, True, True]


@pytest.mark.parametrize("case", FIRST, ids=["%d_to_%d_%dx%d_s%d_f%d" % c[1:7] for c in FIRST])
def test_first_layers(case):
    test_weight_and_bias_gradient(case)


INFINITE = (24, 2, 64, 33, 31)      # B, Cin, Cout, H, W: enough workgroups for the first layers' kernel, 31 pixels a row


def test_an_infinite_frame_value_stays_where_it_is_in_first_layers():
    # the pixel that fills the row's last quad must not multiply the infinite value of the last column by zero
    B, Cin, Cout, H, W = INFINITE
    x = torch.rand((1, B, Cin, H, W), device=DEV)
    x[0, 5, 1, 7, W - 1] = float("inf")
    desc = api.make_desc(1, B, Cin, H, W, Cout, K=1, beta=0.9, theta=1.0, mode=api.TAC_PER_STEP, in_format=REAL)
    v = torch.zeros((1, B, Cout, H, W), device=DEV)
    got = api.tac_conv_lif_backward(desc, x, torch.zeros((Cout, Cin, 3, 3), device=DEV), v, torch.ones_like(v), want_input_grad=False)
    gw = got["grad_w"].cpu()
    assert torch.isfinite(gw[:, 0]).all()
    assert torch.isfinite(gw[:, 1, :, 0]).all() and torch.isinf(gw[:, 1, :, 1:]).all()
