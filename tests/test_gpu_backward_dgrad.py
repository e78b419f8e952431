"""The fp32 matrix-core input gradient at the edges of its tiles: several samples per tile, rows and segments with a
remainder, channel counts that fill no block, the three ways it is written; against the gradient that automatic
differentiation of a double-precision convolution gives for the same dL/dY."""
import numpy as np
import pytest
import torch

from paper_2603_13810_amd import api
from parity_util import np_pack

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
BITS, MEAN, MAX = api.TAC_IN_BITS, api.TAC_IN_BITS_POOL2, api.TAC_IN_BITS_MAXPOOL2

# (B, Cin, Cout, H, W, format, per group, K, T)
CASES = [
    (5, 128, 128, 4, 4, BITS, True, 4, 8),      # several samples per tile, the last tile partly filled
    (3, 5, 3, 1, 1, BITS, False, 2, 5),
    (2, 37, 21, 9, 11, BITS, False, 3, 7),      # weights not readable 16 bytes at a time, two channel blocks
    (1, 130, 9, 6, 70, BITS, True, 2, 3),       # two row segments, two channel groups, rounds of eight with a rest of one
    (2, 72, 40, 16, 16, BITS, True, 4, 6),
    (3, 32, 64, 14, 14, MEAN, False, 4, 7),     # the rate-coded network's second layer
    (2, 20, 16, 5, 40, MAX, False, 2, 3),
    (2, 64, 8, 33, 20, BITS, False, 1, 2),      # strips with a remainder
    (9, 1, 6, 50, 60, BITS, True, 2, 6),        # few input channels over many pixels: the vector kernel, stride 1
    (40, 3, 5, 30, 40, MAX, False, 2, 5),
    (30, 7, 3, 66, 80, MEAN, False, 1, 2),
]
VECTOR = CASES[8:]        # (the choice is held to this on the CPU)


@pytest.mark.parametrize("case", CASES, ids=["%d_to_%d_%dx%d_f%d" % c[1:6] for c in CASES])
def test_input_gradient(case):
    B, Cin, Cout, H, W, fmt, per_group, K, T = case
    r = np.random.Generator(np.random.PCG64(7500 + Cin + Cout + H + W))
    f = 1 if fmt == BITS else 2
    x = (r.random((T, B, Cin, f * H, f * W)) < 0.3).astype(np.uint8)
    desc = api.make_desc(T, B, Cin, H, W, Cout, K=K, beta=0.9, theta=1.0, mode=api.TAC_COLLAPSE, in_format=fmt)
    T_out = api.tac_out_shape(desc)[0]
    v = (0.6 * r.standard_normal((T_out, B, Cout, H, W)) + 0.3).astype(np.float32)
    g = r.standard_normal(v.shape).astype(np.float32)
    w = (r.standard_normal((Cout, Cin, 3, 3)) * 0.1).astype(np.float32)
    got = api.tac_conv_lif_backward(desc, torch.from_numpy(np_pack(x)).to(DEV), torch.from_numpy(w).to(DEV), torch.from_numpy(v).to(DEV),
                                    torch.from_numpy(g).to(DEV), grad_in_per_group=per_group)
    torch.cuda.synchronize()
    gy = got["grad_y"].cpu().double()

    def back(weights, grads):
        a = torch.zeros((T_out * B, Cin, H, W), dtype=torch.float64, requires_grad=True)
        torch.nn.functional.conv2d(a, weights, None, 1, 1).backward(grads.flatten(0, 1))
        return a.grad.view(T_out, B, Cin, H, W).numpy()
    wd = torch.from_numpy(w).double()
    dA, size = back(wd, gy), back(wd.abs(), gy.abs())
    if not per_group:
        beta = float(np.float32(0.9))
        k = np.arange(T) // K
        factor = np.array([beta ** (min(K, T - i // K * K) - 1 - i % K) for i in range(T)])[:, None, None, None, None]
        dA, size = dA[k] * factor, size[k] * factor
        if fmt == MEAN:
            dA, size = (0.25 * a.repeat(2, 3).repeat(2, 4) for a in (dA, size))
        elif fmt == MAX:
            win = x.reshape(T, B, Cin, H, 2, W, 2).transpose(0, 1, 2, 3, 5, 4, 6).reshape(T, B, Cin, H, W, 4)
            first = np.where(win.any(-1), win.argmax(-1), 0)

            def route(a):
                out = np.zeros(win.shape)
                np.put_along_axis(out, first[..., None], a[..., None], -1)
                return out.reshape(T, B, Cin, H, W, 2, 2).transpose(0, 1, 2, 3, 5, 4, 6).reshape(T, B, Cin, 2 * H, 2 * W)
            dA, size = route(dA), route(size)
    # sums of n = 9 Cout fp32 terms in any order and two factors: 2^-24 (sqrt(n) + 3) of the sum of the magnitudes, times four
    tol = 4 * 2.0 ** -24 * ((9 * Cout) ** 0.5 + 3)
    assert (np.abs(got["grad_in"].cpu().numpy() - dA) <= tol * size + 1e-12).all()


def test_an_infinite_weight_of_the_last_channel_is_multiplied_once():
    # five output channels in rounds of eight: the three that fill the round must not multiply the last channel's weights by zero
    B, Cin, Cout, H, W = 1, 6, 5, 6, 6
    desc = api.make_desc(1, B, Cin, H, W, Cout, K=1, beta=0.9, theta=1.0, mode=api.TAC_PER_STEP)
    w = torch.full((Cout, Cin, 3, 3), 0.1, device=DEV)
    w[4, 2, 1, 1] = float("inf")
    v = torch.zeros((1, B, Cout, H, W), device=DEV)
    x = torch.zeros((1, B, Cin, H, 1), dtype=torch.int32, device=DEV)
    got = api.tac_conv_lif_backward(desc, x, w, v, torch.ones_like(v))["grad_in"][0, 0]
    assert (got[2] == float("inf")).all()             # the centre tap meets every pixel's own dL/dY, which is positive
    others = [0, 1, 3, 4, 5]
    assert torch.isfinite(got[others]).all() and (got[others] > 0).all()


# Many tiles: products of bf16 thirds, (B, Cin, Cout, H, W, format, per group, K, T) as above
MANY = [
    (70, 33, 8, 9, 33, BITS, True, 2, 4),       # one round; two channel groups, the second of one channel
    (70, 33, 9, 9, 33, BITS, True, 2, 4),       # one round, half of it but for one channel empty
    (60, 40, 17, 16, 16, BITS, True, 1, 2),     # a second round of one channel
    (20, 64, 32, 21, 65, BITS, False, 2, 3),    # two row segments, the second of one pixel
    (300, 96, 24, 6, 5, BITS, True, 2, 2),      # several samples a tile, the last tile partly filled
    (90, 32, 64, 14, 14, MEAN, False, 4, 7),
    (40, 24, 40, 11, 30, MAX, False, 2, 3),
    (70, 33, 1, 9, 33, BITS, False, 2, 4),      # up to eight output channels: two taps a product
    (50, 70, 7, 20, 45, BITS, True, 2, 3), (3, 40, 8, 5, 5, BITS, True, 2, 3), (90, 24, 5, 14, 14, MEAN, False, 4, 7), (40, 24, 3, 11, 30, MAX, False, 2, 3),
]


@pytest.mark.parametrize("case", MANY, ids=["%d_to_%d_%dx%d_f%d" % c[1:6] for c in MANY])
def test_input_gradient_on_many_tiles(case):
    test_input_gradient(case)


def test_values_that_have_no_thirds():
    # infinities, NaN, a value that rounds beyond the largest bf16, subnormal ones
    B, Cin, Cout, H, W = 60, 40, 24, 16, 16
    r = np.random.Generator(np.random.PCG64(7600))
    desc = api.make_desc(1, B, Cin, H, W, Cout, K=1, beta=0.9, theta=1.0, mode=api.TAC_PER_STEP)
    v = np.full((1, B, Cout, H, W), 1.0, np.float32)                # at the threshold: the surrogate's factor is 1
    g = r.standard_normal(v.shape).astype(np.float32)
    g[0, 1, 3, 5, 5] = np.inf
    g[0, 2, 20, 0, 15] = -np.inf
    g[0, 3, 0, 8, 8], g[0, 3, 1, 8, 9] = np.inf, -np.inf
    g[0, 4, 23, 15, 0] = np.nan
    g[0, 5, 7, 4, 4] = 3.4e38
    g[0, 6] = 0.0
    g[0, 6, 5, 5, 5] = 1e-40
    w = (r.standard_normal((Cout, Cin, 3, 3)) * 0.1).astype(np.float32)
    x = np_pack((r.random((1, B, Cin, H, W)) < 0.3).astype(np.uint8))
    got = api.tac_conv_lif_backward(desc, torch.from_numpy(x).to(DEV), torch.from_numpy(w).to(DEV), torch.from_numpy(v).to(DEV), torch.from_numpy(g).to(DEV),
                                    grad_in_per_group=True)
    torch.cuda.synchronize()
    gy = got["grad_y"].cpu().double()[0]
    assert gy.isinf().sum() == 4 and gy.isnan().sum() == 1

    def back(weights, grads):
        return torch.nn.functional.conv_transpose2d(grads, weights, padding=1).numpy()
    wd = torch.from_numpy(w).double()
    have, want = got["grad_in"].cpu().numpy().reshape(B, Cin, H, W), back(wd, gy)
    assert np.array_equal(np.isnan(have), np.isnan(want))
    inf = np.isinf(want)
    assert inf.any() and np.array_equal(have[inf], want[inf].astype(np.float32))
    ok = np.isfinite(want)
    size = back(wd.abs(), gy.nan_to_num(0.0, 0.0, 0.0).abs())
    # the bound above, and 2^-126 per product of a subnormal part that the matrix cores may take as zero
    tol = 4 * 2.0 ** -24 * ((9 * Cout) ** 0.5 + 3)
    assert (np.abs(have[ok] - want[ok]) <= tol * size[ok] + 9 * Cout * 2.0 ** -126).all()


@pytest.mark.parametrize("Cout", [1, 7, 8])
def test_values_that_have_no_thirds_in_one_round(Cout):
    # up to eight output channels: a product takes two taps, the last one with zeros in the place of a tenth
    B, Cin, H, W = 60, 40, 16, 16
    r = np.random.Generator(np.random.PCG64(7650 + Cout))
    desc = api.make_desc(1, B, Cin, H, W, Cout, K=1, beta=0.9, theta=1.0, mode=api.TAC_PER_STEP)
    g = r.standard_normal((1, B, Cout, H, W)).astype(np.float32)
    last = Cout - 1
    g[0, 1, last, 5, 5], g[0, 2, 0, 0, 15], g[0, 3, last, 15, 0], g[0, 4, last, 7, 7] = np.inf, -np.inf, np.inf, np.nan
    w = (r.standard_normal((Cout, Cin, 3, 3)) * 0.1).astype(np.float32)
    x = torch.zeros((1, B, Cin, H, 1), dtype=torch.int32, device=DEV)
    gd = torch.from_numpy(g).to(DEV)
    got = api.tac_conv_lif_backward(desc, x, torch.from_numpy(w).to(DEV), torch.ones_like(gd), gd, grad_in_per_group=True)
    gy, wd = got["grad_y"].cpu().double()[0], torch.from_numpy(w).double()
    have, want = got["grad_in"].cpu().numpy().reshape(B, Cin, H, W), torch.nn.functional.conv_transpose2d(gy, wd, padding=1).numpy()
    assert np.array_equal(np.isnan(have), np.isnan(want)) and np.isinf(want).any()
    assert np.array_equal(have[np.isinf(want)], want[np.isinf(want)].astype(np.float32))
    ok = np.isfinite(want)
    size = torch.nn.functional.conv_transpose2d(gy.nan_to_num(0.0, 0.0, 0.0).abs(), wd.abs(), padding=1).numpy()
    assert (np.abs(have[ok] - want[ok]) <= 4 * 2.0 ** -24 * ((9 * Cout) ** 0.5 + 3) * size[ok]).all()


def test_planes_beyond_one_descriptor():
    # 2^23 pixels and more: every channel of a round has a descriptor of its own; corners and a middle part against double precision
    Cin, Cout, H, W = 20, 18, 8397, 1000
    desc = api.make_desc(1, 1, Cin, H, W, Cout, K=1, beta=0.9, theta=1.0, mode=api.TAC_PER_STEP)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(76)
    g = torch.randn((1, 1, Cout, H, W), generator=gen, device=DEV)
    w = torch.randn((Cout, Cin, 3, 3), generator=gen, device=DEV) * 0.1
    x = torch.zeros((1, 1, Cin, H, (W + 31) // 32), dtype=torch.int32, device=DEV)
    got = api.tac_conv_lif_backward(desc, x, w, torch.ones_like(g), g, grad_in_per_group=True)
    torch.cuda.synchronize()
    gy, have = got["grad_y"][0, 0], got["grad_in"].view(Cin, H, W)
    wd, pad = w.cpu().double(), torch.nn.functional.pad
    tol = 4 * 2.0 ** -24 * ((9 * Cout) ** 0.5 + 3)
    for y0, x0 in ((0, 0), (0, W - 70), (H - 20, 0), (H - 20, W - 70), (4450, 500)):
        y1, x1 = min(y0 + 20, H), min(x0 + 70, W)
        part = pad(gy[:, max(y0 - 1, 0):y1 + 1, max(x0 - 1, 0):x1 + 1].cpu().double(), (int(x0 == 0), int(x1 == W), int(y0 == 0), int(y1 == H)))
        # a part with a ring of one around it: the transposed convolution loses the ring on either side
        want = torch.nn.functional.conv_transpose2d(part[None], wd, padding=2)[0]
        size = torch.nn.functional.conv_transpose2d(part[None].abs(), wd.abs(), padding=2)[0]
        assert want.shape[1:] == (y1 - y0, x1 - x0)
        assert ((have[:, y0:y1, x0:x1].cpu().double() - want).abs() <= tol * size + 1e-12).all()


@pytest.mark.parametrize("Cout", [1, 2, 4, 8, 24])
def test_few_output_channels_are_no_further_off_than_products_of_fp32(Cout):
    # 400 tiles: products of bf16 thirds.  What products of fp32 leave is put together here, two output channels and a tap at a time, each sum rounded to fp32.
    B, Cin, H, W = 100, 40, 28, 28
    gen = torch.Generator(device=DEV)
    gen.manual_seed(7700 + Cout)
    desc = api.make_desc(1, B, Cin, H, W, Cout, K=1, beta=0.9, theta=1.0, mode=api.TAC_PER_STEP)
    g = torch.randn((1, B, Cout, H, W), generator=gen, device=DEV)
    w = torch.randn((Cout, Cin, 3, 3), generator=gen, device=DEV) * 0.1
    x = torch.zeros((1, B, Cin, H, 1), dtype=torch.int32, device=DEV)
    got = api.tac_conv_lif_backward(desc, x, w, torch.ones_like(g), g, grad_in_per_group=True)
    have = got["grad_in"].view(B, Cin, H * W)
    gy, wd = torch.nn.functional.pad(got["grad_y"][0].double(), (1, 1, 1, 1)), w.double()
    want = torch.zeros((B, Cin, H * W), dtype=torch.float64, device=DEV)
    fp32 = torch.zeros((B, Cin, H * W), device=DEV)
    for co in range(0, Cout, 2):
        for tap in range(9):
            ky, kx = 2 - tap // 3, 2 - tap % 3
            seen = gy[:, co:co + 2, ky:ky + H, kx:kx + W]
            add = (wd[co:co + 2, None, :, tap // 3, tap % 3, None] * seen.reshape(B, -1, 1, H * W).transpose(0, 1)).sum(0)
            want += add
            fp32 = (fp32.double() + add).float()
    err, err32 = (have.double() - want).norm(), (fp32.double() - want).norm()
    print("Cout", Cout, "error", float(err / want.norm()), "of products of fp32", float(err32 / want.norm()))
    assert err <= err32


@pytest.mark.parametrize("shift_g,shift_w", [(-118, 0), (-60, -62), (0, -118), (-95, 0)])
def test_tiny_values_keep_their_digits(shift_g, shift_w):
    # thirds of values below 2^-110 reach below the smallest subnormal bf16
    B, Cin, Cout, H, W = 60, 40, 24, 16, 16
    r = np.random.Generator(np.random.PCG64(7800))
    desc = api.make_desc(1, B, Cin, H, W, Cout, K=1, beta=0.9, theta=1.0, mode=api.TAC_PER_STEP)
    g = np.ldexp(r.standard_normal((1, B, Cout, H, W)), shift_g).astype(np.float32)
    g[0, B // 2:] *= np.float32(0.0)
    w = np.ldexp(r.standard_normal((Cout, Cin, 3, 3)), shift_w).astype(np.float32)
    x = torch.zeros((1, B, Cin, H, 1), dtype=torch.int32, device=DEV)
    gd = torch.from_numpy(g).to(DEV)
    got = api.tac_conv_lif_backward(desc, x, torch.from_numpy(w).to(DEV), torch.ones_like(gd), gd, grad_in_per_group=True)
    gy, wd = got["grad_y"].cpu().double()[0], torch.from_numpy(w).double()
    want, size = (torch.nn.functional.conv_transpose2d(a, b, padding=1) for a, b in ((gy, wd), (gy.abs(), wd.abs())))
    # the bound of the other tests, and half of the smallest subnormal number for each rounding of a sum
    tol = 4 * 2.0 ** -24 * ((9 * Cout) ** 0.5 + 3)
    assert ((got["grad_in"].cpu().double().view_as(want) - want).abs() <= tol * size + 9 * Cout * 2.0 ** -150).all()


@pytest.mark.parametrize("Cin,fmt,per_group", [((1 << 20) + 5, BITS, False), (1 << 20, BITS, True), ((1 << 20) + 2, MEAN, False)])
def test_more_input_channels_than_a_grid_has_rows_for(Cin, fmt, per_group):
    # the vector kernel's channels go on in x
    B, Cout, H, W, T = 1, 2, 2, 2, 1
    gen = torch.Generator(device=DEV)
    gen.manual_seed(79)
    desc = api.make_desc(T, B, Cin, H, W, Cout, K=1, beta=0.9, theta=1.0, mode=api.TAC_PER_STEP, in_format=fmt)
    f = 1 if fmt == BITS else 2
    g = torch.randn((T, B, Cout, H, W), generator=gen, device=DEV)
    w = torch.randn((Cout, Cin, 3, 3), generator=gen, device=DEV) * 0.1
    x = torch.zeros((T, B, Cin, f * H, 1), dtype=torch.int32, device=DEV)
    got = api.tac_conv_lif_backward(desc, x, w, torch.ones_like(g), g, grad_in_per_group=per_group)
    gy, wd = got["grad_y"][0].cpu().double(), w.cpu().double()
    want, size = (torch.nn.functional.conv_transpose2d(a, b, padding=1).view(Cin, H, W) for a, b in ((gy, wd), (gy.abs(), wd.abs())))
    if fmt == MEAN:
        want, size = (0.25 * a.repeat_interleave(2, 1).repeat_interleave(2, 2) for a in (want, size))
    tol = 4 * 2.0 ** -24 * ((9 * Cout) ** 0.5 + 3)
    assert ((got["grad_in"].cpu().double().view_as(want) - want).abs() <= tol * size + 1e-12).all()
