"""The in-between matrix-core kernel at the edges of its tiles: pixel blocks of 1 to 16 rows, tiles that straddle samples,
partial tiles in rows and channels, groups of up to 32 frames, every way to load, and a shorter last group inside the
launch; against the oracle."""
import numpy as np
import pytest
import torch

from paper_2603_13810_amd import api, synth
from gpu_util import check_layer

pytestmark = pytest.mark.gpu
B16, F32 = api.TAC_BF16, api.TAC_FP32
TAC, TP, STEP = api.TAC_COLLAPSE, api.TAC_PRESERVE, api.TAC_PER_STEP

# (B, Cin, Cout, H, W, stride, pool on load, pool in the writer, precision, mode, K, T)
CASES = [
    (3, 8, 5, 1, 1, 1, False, False, B16, TAC, 2, 5),                 # one pixel, sixteen rows of two lanes per block
    (5, 8, 33, 3, 2, 1, False, False, B16, TP, 3, 7),                 # tiles straddle the samples; a second channel block of one
    (7, 128, 40, 4, 4, 1, False, True, B16, TP, 4, 8),                # the deep blocks of the event-data network
    (5, 128, 128, 2, 2, 1, False, True, B16, TAC, 2, 4),
    (3, 40, 70, 9, 13, 1, False, False, B16, TAC, 4, 11),             # 16 lanes a row, parts of rows per wave
    (2, 48, 80, 11, 45, 1, False, False, B16, TAC, 4, 9),             # two words a row
    (2, 24, 36, 6, 20, 1, False, True, B16, TP, 2, 5),                # pooled rows across a wave's two blocks
    (2, 24, 36, 6, 40, 1, False, True, B16, TAC, 8, 17),              # the same with two words a row
    (1, 56, 20, 7, 61, 2, False, False, B16, TAC, 16, 33),            # stride 2, two chunks of frames, one frame left over
    (1, 16, 40, 5, 100, 2, True, False, B16, TP, 5, 12),              # stride 2 behind the mean pool, 200 stored pixels
    (2, 32, 64, 14, 14, 1, True, False, B16, TAC, 17, 35),            # mean pool, three chunks of frames
    (2, 24, 17, 8, 10, 1, "max", False, B16, TAC, 3, 8),
    (1, 16, 33, 6, 36, 1, "max", False, B16, TP, 32, 40),             # max pool, four chunks of frames
    (3, 64, 48, 7, 7, 1, False, False, F32, TAC, 4, 10),
    (2, 32, 64, 14, 14, 1, True, False, F32, TAC, 8, 25),             # the rate-coded network's second layer, 25 frames
    (2, 16, 40, 9, 33, 2, "max", False, F32, STEP, 1, 3),
    (2, 8, 24, 6, 40, 1, False, True, F32, TAC, 2, 4),
    (3, 8, 80, 17, 16, 1, False, False, B16, STEP, 1, 5),             # single frames: bits as they are, mean pool, max pool
    (2, 24, 40, 9, 21, 1, True, False, B16, STEP, 1, 4),
    (2, 40, 24, 6, 18, 1, "max", True, B16, STEP, 1, 3),
    (1, 32, 40, 7, 9, 2, True, False, F32, STEP, 1, 3),
]

# The tile is chosen by its estimated time, and layers as small as those above take the smallest one.  These take the other
# variants: the launch's plan has the values named here, without the membrane trace and with it (where only the first is
# named the second differs).  test_mid_plan.py holds the choice to them on the CPU.
VARIANTS = {
    "two channel blocks": ((1, 80, 40, 3, 37, 2, True, False, B16, TAC, 2, 4), dict(nmc=2, nnp=1, direct=0)),
    "two by two blocks, one with the trace": ((16, 8, 200, 19, 19, 1, "max", False, B16, TAC, 4, 6), dict(nmc=2, nnp=2, direct=0), dict(nmc=2, nnp=1)),
    "two by two blocks": ((40, 8, 200, 30, 33, 1, False, False, B16, TP, 4, 5), dict(nmc=2, nnp=2, direct=0)),
    "two by two blocks, direct": ((40, 8, 200, 11, 34, 1, False, False, B16, STEP, 1, 3), dict(nmc=2, nnp=2, direct=1)),
    "eight jobs": ((1, 96, 40, 7, 3, 1, "max", False, B16, TAC, 2, 3), dict(jobs=8, batches=1)),
    "two batches": ((1, 112, 96, 7, 2, 1, True, False, B16, TAC, 2, 5), dict(jobs=4, batches=2)),
    "eight jobs of two batches": ((1, 120, 96, 20, 2, 2, "max", False, B16, STEP, 1, 2), dict(jobs=8, batches=2)),
    "two loaders, fp32": ((1, 112, 70, 10, 2, 2, "max", False, F32, TAC, 8, 17), dict(loaders=2)),
    "two loaders of two batches": ((1, 48, 70, 3, 119, 2, True, True, B16, TAC, 32, 33), dict(loaders=2, batches=2)),
    "two channel blocks, direct": ((16, 8, 200, 19, 33, 1, False, False, B16, STEP, 1, 3), dict(nmc=2, nnp=1, direct=1)),
    "direct, tiles that straddle samples": ((24, 8, 200, 3, 20, 1, False, False, B16, STEP, 1, 3), dict(direct=1, flatten=1, rpb=1)),
    "direct, blocks that straddle samples": ((32, 8, 130, 3, 9, 1, False, False, B16, STEP, 1, 3), dict(direct=1, flatten=1, rpb=2)),
    "direct, two rows a block, a last group of one": ((3, 16, 70, 9, 14, 1, False, False, B16, TP, 2, 5), dict(direct=1, rpb=2)),
    "direct, fp32, stride 2": ((2, 24, 33, 6, 30, 2, False, False, F32, TAC, 2, 7), dict(direct=1)),
    "direct, max pool, pooled output": ((2, 8, 33, 12, 20, 1, "max", True, B16, STEP, 1, 3), dict(direct=1, nnp=2)),
    "direct, two pixels a thread": ((3, 24, 20, 17, 30, 1, False, False, B16, TAC, 2, 3), dict(direct=1, flatten=0)),
    "direct, mean pool, fp32": ((3, 16, 24, 18, 40, 1, True, False, F32, STEP, 1, 2), dict(direct=1)),
    "direct, eight rows a block, fp32, stride 2": ((3, 32, 48, 7, 7, 2, "max", False, F32, STEP, 1, 2), dict(direct=1, rpb=8)),
}


def _check(case):
    B, Cin, Cout, H, W, stride, pool, out_pool, precision, mode, K, T = case
    r = np.random.Generator(np.random.PCG64(6000 + Cin + Cout + H + W + K))
    f = 2 if pool else 1
    s = (r.random((T, B, Cin, f * H, f * W)) < 0.12).astype(np.uint8)
    w = synth.kaiming_normal(61, Cout, Cin) * np.float32(1.5)
    bias = (r.standard_normal(Cout) * 0.1).astype(np.float32)
    Ho, Wo = (H - 1) // stride + 1, (W - 1) // stride + 1
    v0 = (r.standard_normal((B, Cout, Ho, Wo)) * 0.3).astype(np.float32)
    samples = dict(oracle_samples=[0, 1, B // 2, B - 1]) if B > 8 else {}
    par, g, ref = check_layer(s, w, K=K, beta=0.9, theta=1.0, mode=mode, stride=stride, pool2=pool, precision=precision, bias=bias,
                              v0=v0, expect_kernel=api.TAC_KERNEL_MFMA, **(dict(out_pool=True) if out_pool else {}), **samples)
    assert ref[0].any()
    print(case, par)


@pytest.mark.parametrize("case", CASES, ids=["%dx%d_to_%d_%dx%d_K%d" % (c[0], c[1], c[2], c[3], c[4], c[10]) for c in CASES])
def test_edges_of_the_tiles(case):
    _check(case)


@pytest.mark.parametrize("name", VARIANTS)
def test_variants_of_the_tile(name):
    _check(VARIANTS[name][0])


def test_last_rows_of_a_very_tall_image():
    # 217 million neurons a channel: byte offsets of the fifth channel's last rows do not fit 32 bits.  What the layer leaves in its
    # first and last rows is what it leaves for an image of those rows alone.
    H, W, C, part = 3_400_000, 64, 8, 80
    dev = "cuda:0"
    gen = torch.Generator(device=dev)
    gen.manual_seed(11)
    frames = torch.randint(-2 ** 31, 2 ** 31 - 1, (1, 1, C, H, W // 32), dtype=torch.int32, device=dev, generator=gen)
    frames &= torch.randint(-2 ** 31, 2 ** 31 - 1, frames.shape, dtype=torch.int32, device=dev, generator=gen)
    w = torch.from_numpy(synth.kaiming_normal(67, C, C)).to(dev)

    def run(x):
        desc = api.make_desc(1, 1, C, x.shape[3], W, C, K=1, beta=0.9, theta=0.5, mode=STEP, precision=B16)
        assert api.tac_select_kernel(desc) == api.TAC_KERNEL_MFMA
        v = torch.zeros((1, C, x.shape[3], W), dtype=torch.float32, device=dev)
        return api.tac_conv_lif(desc, x, api.tac_prepare_weights(desc, w), None, v), v
    spikes, v = run(frames)
    for rows, inner in ((slice(0, part), slice(0, part - 1)), (slice(H - part, H), slice(1, part))):
        spikes_part, v_part = run(frames[:, :, :, rows].contiguous())
        assert spikes_part.any()
        assert torch.equal(spikes[:, :, :, rows][:, :, :, inner], spikes_part[:, :, :, inner])
        assert torch.equal(v[:, :, rows][:, :, inner], v_part[:, :, inner])
