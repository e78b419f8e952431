"""Small images on many channels in the in-between kernel: eight waves share a workgroup's pixel blocks, eight or four of them one,
and add up their parts of the contraction; against the oracle, at the edges of the ranges of k-steps, of the blocks and of the four
steps that are stored together."""
import numpy as np
import pytest

from paper_2603_13810_amd import api, synth
from gpu_util import check_layer

pytestmark = pytest.mark.gpu
TAC, TP, STEP = api.TAC_COLLAPSE, api.TAC_PRESERVE, api.TAC_PER_STEP

# (B, Cin, Cout, H, W, stride, pool in the writer, mode, K, T, what)
CASES = [
    (1, 64, 32, 1, 1, 1, False, TAC, 2, 3, "one pixel, ranges of four and five steps"),
    (2, 64, 33, 2, 2, 1, True, TP, 3, 7, "a second block of one channel, three steps together, a last group of one"),
    (3, 72, 40, 3, 16, 1, False, TP, 5, 11, "five steps in two goes, rows of 16"),
    (5, 96, 64, 7, 7, 1, False, TAC, 4, 9, "blocks that straddle samples"),
    (16, 128, 128, 16, 16, 1, True, TP, 4, 8, "four waves a block"),
    (16, 128, 128, 4, 4, 1, True, TP, 8, 16, "eight waves a block, eight steps"),
    (1, 128, 70, 16, 9, 1, False, STEP, 1, 3, "single frames"),
    (4, 120, 48, 12, 10, 1, False, TP, 2, 5, "groups of two, fewer waves than channel groups"),
    (2, 80, 96, 9, 31, 2, False, TAC, 16, 33, "stride 2, two chunks of frames, one frame left over"),
    (1, 104, 130, 15, 3, 2, False, TP, 32, 40, "groups of 32"),
]


@pytest.mark.parametrize("case", CASES, ids=[c[-1] for c in CASES])
def test_waves_that_share_a_pixel_block(case):
    B, Cin, Cout, H, W, stride, out_pool, mode, K, T, _ = case
    r = np.random.Generator(np.random.PCG64(6600 + Cin + Cout + H + W + K))
    s = (r.random((T, B, Cin, H, W)) < 0.12).astype(np.uint8)
    w = synth.kaiming_normal(63, Cout, Cin) * np.float32(1.5)
    bias = (r.standard_normal(Cout) * 0.1).astype(np.float32)
    Ho, Wo = (H - 1) // stride + 1, (W - 1) // stride + 1
    v0 = (r.standard_normal((B, Cout, Ho, Wo)) * 0.3).astype(np.float32)
    par, g, ref = check_layer(s, w, K=K, beta=0.9, theta=1.0, mode=mode, stride=stride, precision=api.TAC_BF16, bias=bias, v0=v0,
                              expect_kernel=api.TAC_KERNEL_MFMA, **(dict(out_pool=True) if out_pool else {}),
                              **(dict(oracle_samples=[0, 1, B - 1]) if B > 8 else {}))
    assert ref[0].any()
    print(case, par)


# fp32 layers: two tiles of 32 output channels over one aggregate tile; a last workgroup with one of them, a tile of few channels
@pytest.mark.parametrize("case", [(2, 32, 96, 9, 14, 1, True, TAC, 4, 9), (1, 16, 33, 7, 20, 2, False, TP, 3, 7), (3, 40, 130, 5, 6, 1, False, TAC, 16, 17)],
                         ids=["three tiles", "a second tile of one channel", "five tiles, a last group of one"])
def test_two_channel_tiles_over_one_aggregate_tile_fp32(case):
    B, Cin, Cout, H, W, stride, pool, mode, K, T = case
    r = np.random.Generator(np.random.PCG64(6700 + Cin + Cout + K))
    f = 2 if pool else 1
    s = (r.random((T, B, Cin, f * H, f * W)) < 0.12).astype(np.uint8)
    w = synth.kaiming_normal(64, Cout, Cin) * np.float32(1.5)
    bias = (r.standard_normal(Cout) * 0.1).astype(np.float32)
    Ho, Wo = (H - 1) // stride + 1, (W - 1) // stride + 1
    v0 = (r.standard_normal((B, Cout, Ho, Wo)) * 0.3).astype(np.float32)
    par, g, ref = check_layer(s, w, K=K, beta=0.9, theta=1.0, mode=mode, stride=stride, pool2=pool, precision=api.TAC_FP32, bias=bias, v0=v0,
                              expect_kernel=api.TAC_KERNEL_MFMA)
    assert ref[0].any()
    print(case, par)
