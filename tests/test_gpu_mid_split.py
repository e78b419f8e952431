"""Small images on many channels in the in-between kernel: eight waves share a workgroup's pixel blocks, eight or four of them one,
and add up their parts of the contraction; against the oracle, at the edges of the ranges of k-steps, of the blocks and of the four
steps that are stored together.  And fp32 layers of several tiles of 32 output channels, one or two tiles a workgroup."""
import numpy as np
import pytest

from paper_2603_13810_amd import api, synth
from gpu_util import check_layer, run_gpu
from parity_util import TOL_FP32, compare

pytestmark = pytest.mark.gpu
B16, F32 = api.TAC_BF16, api.TAC_FP32
TAC, TP, STEP = api.TAC_COLLAPSE, api.TAC_PRESERVE, api.TAC_PER_STEP

# (B, Cin, Cout, H, W, stride, pool in the writer, mode, K, T, what)
CASES = [
    (1, 64, 32, 1, 1, 1, False, TAC, 2, 3, "one pixel, ranges of four and five steps"),
    (2, 64, 33, 2, 2, 1, True, TP, 3, 7, "a second block of one channel, three steps together, a last group of one"),
    (3, 72, 40, 3, 16, 1, False, TP, 5, 11, "five steps in two goes, rows of 16"),
    (5, 96, 64, 7, 7, 1, False, TAC, 4, 9, "rows of seven pixels"),
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


# fp32 layers of so few rows that a workgroup takes one tile of 32 output channels; the last tile has few channels
@pytest.mark.parametrize("case", [(2, 32, 96, 9, 14, 1, True, TAC, 4, 9), (1, 16, 33, 7, 20, 2, False, TP, 3, 7), (3, 40, 130, 5, 6, 1, False, TAC, 16, 17)],
                         ids=["three tiles", "a second tile of one channel", "five tiles, a last group of one"])
def test_one_channel_tile_over_an_aggregate_tile_fp32(case):
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


# (B, Cin, Cout, H, W, stride, pool on load, pool in the writer, precision, mode, K, T), and what the launch's plan has in it, with and
# without the membrane trace (test_mid_plan.py holds the choice to it on the CPU).  nco = 2: two tiles of 32 output channels over one
# aggregate tile, the last workgroup of an odd number with one of them.
VARIANTS = {
    "fp32, two tiles a workgroup, three in all, stride 2": ((2, 24, 96, 10, 15, 2, True, False, F32, TAC, 16, 32), dict(nco=2)),
    "fp32, a second tile of one channel, two words a row": ((20, 32, 33, 18, 47, 1, "max", False, F32, TAC, 2, 5), dict(nco=2, rpb=1)),
    "fp32, five tiles, two words a row": ((12, 32, 130, 9, 35, 1, True, False, F32, TAC, 4, 9), dict(nco=2, rpb=1)),
    "fp32, five tiles, blocks of two samples": ((32, 40, 160, 17, 9, 1, True, False, F32, TAC, 3, 7), dict(nco=2, flatten=1, rpb=2)),
    "fp32, three tiles, two loaders": ((32, 48, 96, 6, 48, 1, "max", False, F32, TAC, 8, 9), dict(nco=2, loaders=2)),
    "fp32, five tiles, pooled output": ((20, 40, 160, 24, 12, 1, False, True, F32, TAC, 2, 5), dict(nco=2)),
    "fp32, three tiles, a last group of one": ((64, 32, 96, 14, 14, 1, True, False, F32, TP, 3, 7), dict(nco=2, rpb=2)),
    "eight waves a block of two samples, two jobs a wave": ((2, 104, 33, 19, 2, 1, False, False, B16, TP, 4, 9), dict(split=8, flatten=1, rpb=16, jobs=13, batches=1)),
    "eight waves a block, two batches, stride 2": ((2, 88, 130, 15, 1, 2, False, False, B16, TP, 5, 6), dict(split=8, batches=2)),
    "four waves a block of two samples, direct": ((12, 72, 96, 15, 13, 1, False, False, B16, TP, 2, 5), dict(split=4, flatten=1, rpb=2, direct=1)),
    "four waves a block, two jobs of two batches": ((64, 104, 130, 14, 1, 1, False, False, B16, TAC, 3, 4), dict(split=4, flatten=1, jobs=13, batches=2)),
}


@pytest.mark.parametrize("name", VARIANTS)
def test_variant(name):
    B, Cin, Cout, H, W, stride, pool, out_pool, precision, mode, K, T = VARIANTS[name][0]
    r = np.random.Generator(np.random.PCG64(6800 + Cin + Cout + H + W + K))
    f = 2 if pool else 1
    s = (r.random((T, B, Cin, f * H, f * W)) < 0.12).astype(np.uint8)
    w = synth.kaiming_normal(65, Cout, Cin) * np.float32(1.5)
    bias = (r.standard_normal(Cout) * 0.1).astype(np.float32)
    Ho, Wo = (H - 1) // stride + 1, (W - 1) // stride + 1
    v0 = (r.standard_normal((B, Cout, Ho, Wo)) * 0.3).astype(np.float32)
    par, g, ref = check_layer(s, w, K=K, beta=0.9, theta=1.0, mode=mode, stride=stride, pool2=pool, precision=precision, bias=bias, v0=v0,
                              expect_kernel=api.TAC_KERNEL_MFMA, oracle_samples=[0, 1, B // 2, B - 1] if B > 8 else None,
                              **(dict(out_pool=True) if out_pool else {}))
    assert ref[0].any()
    print(name, par)


# (samples of a call whose waves share blocks, samples of one whose waves do not), 128 -> 128 channels at 16 x 16
SHARED, ALONE = (8, 16), (32, 64)


def test_a_batch_and_its_parts_agree():
    """The rule for sharing blocks looks at the batch, and the two sides of it sum in different orders: a batch agrees with its parts to the
    precision of fp32 sums, and bit for bit where both are on one side."""
    r = np.random.Generator(np.random.PCG64(6900))
    s = (r.random((8, 64, 128, 16, 16)) < 0.12).astype(np.uint8)
    w = synth.kaiming_normal(66, 128, 128) * np.float32(1.5)
    bias = (r.standard_normal(128) * 0.1).astype(np.float32)
    kw = dict(K=4, beta=0.9, theta=1.0, mode=TP, precision=B16, bias=bias)
    runs = {B: [run_gpu(s[:, i:i + B], w, **kw) for i in range(0, 64, B)] for B in SHARED + ALONE}
    spikes, traces = ({B: np.concatenate([g[k] for g in v], axis=1) for B, v in runs.items()} for k in ("spikes", "v_trace"))
    for one, other in (SHARED, ALONE):
        assert np.array_equal(spikes[one], spikes[other]) and np.array_equal(traces[one], traces[other])
    par = compare(spikes[SHARED[1]], traces[SHARED[1]].astype(np.float64), spikes[ALONE[0]], traces[ALONE[0]], 1.0, TOL_FP32)
    assert par.ok, par
    print("a batch and its parts", par)
