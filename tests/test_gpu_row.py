"""bf16 layers of up to 128 channels on the row kernel (17 to 64 output pixels a row, no pool, membranes not recorded): against the oracle, and bit for bit
against the kernel that takes the same layer when its membranes are recorded."""
import numpy as np
import pytest

from paper_2603_13810_amd import api, synth
from gpu_util import check_layer, run_gpu

pytestmark = pytest.mark.gpu
TAC, TP, STEP = api.TAC_COLLAPSE, api.TAC_PRESERVE, api.TAC_PER_STEP

# (B, Cin, Cout, H, W, stride, mode, K, T, what, what the launch's plan has in it: test_row_plan.py holds the choice to it on the CPU)
CASES = [
    (1, 24, 32, 3, 17, 1, STEP, 1, 3, "rows of 17, three jobs for four waves", dict(kp=1, spr=2, n_jobs=3, waves=4)),
    (3, 40, 40, 9, 30, 1, TAC, 2, 9, "a last group of one, a last tile of eight channels, a job of one block", dict(kp=2, cb=4, n_jobs=4, co_tiles=2)),
    (2, 56, 24, 6, 64, 1, TAC, 4, 7, "rows of 64, a last group of three, waves that only load", dict(kp=4, spr=4, pw=2, waves=6)),
    (4, 48, 80, 45, 45, 1, TAC, 4, 9, "an odd number of segments, three tiles of channels", dict(spr=3, nco=3, nnp=1)),
    (2, 128, 128, 10, 33, 1, TP, 8, 17, "groups of eight, one frame left over, all the channels", dict(kp=8, nks=72)),
    (3, 32, 70, 12, 21, 1, TAC, 16, 33, "two tables, one frame left over", dict(kp=16, spr=2)),
    (2, 24, 32, 8, 48, 1, TP, 12, 26, "groups of twelve, the last of two", dict(kp=16, spr=3)),
    (2, 40, 100, 13, 127, 2, TAC, 5, 11, "stride 2, rows of 127", dict(kp=8, spr=4)),
    (3, 72, 64, 11, 34, 2, STEP, 1, 5, "stride 2, rows of 17", dict(kp=1, spr=2)),
    (16, 128, 128, 28, 28, 1, TP, 4, 5, "seven rows a tile, three turns of jobs", dict(pw=7, tr=7, n_jobs=24)),
    (24, 8, 200, 20, 60, 1, TAC, 3, 4, "two blocks a wave, a last tile of one block of channels", dict(kp=4, nnp=2, nco=2, co_tiles=4)),
    (30, 64, 64, 20, 49, 1, TAC, 8, 9, "twelve waves, a last tile of two rows", dict(kp=8, pw=6, nco=2, tr=3)),
    (300, 8, 16, 5, 18, 1, TP, 3, 6, "tiles that straddle samples", dict(flatten=1, tr=6)),
    (60, 16, 128, 13, 33, 1, TAC, 16, 32, "two blocks a wave, an odd number of segments", dict(kp=16, nnp=2, spr=3)),
    (60, 64, 128, 13, 33, 1, TAC, 2, 4, "groups of two, two blocks a wave", dict(kp=2, nnp=2)),
]


@pytest.mark.parametrize("case", CASES, ids=[c[-2] for c in CASES])
def test_layer(case):
    B, Cin, Cout, H, W, stride, mode, K, T = case[:9]
    r = np.random.Generator(np.random.PCG64(7300 + Cin + Cout + H + W + K))
    s = (r.random((T, B, Cin, H, W)) < 0.12).astype(np.uint8)
    w = synth.kaiming_normal(73, Cout, Cin) * np.float32(1.5)
    bias = (r.standard_normal(Cout) * 0.1).astype(np.float32)
    Ho, Wo = (H - 1) // stride + 1, (W - 1) // stride + 1
    v0 = (r.standard_normal((B, Cout, Ho, Wo)) * 0.3).astype(np.float32)
    kw = dict(K=K, beta=0.9, theta=1.0, mode=mode, stride=stride, precision=api.TAC_BF16, bias=bias, v0=v0)
    # (it runs the layer with and without recorded membranes, and the bits and final membranes of the two have to be the same)
    par, _, ref = check_layer(s, w, expect_kernel=api.TAC_KERNEL_MFMA, **kw, **(dict(oracle_samples=[0, B - 1]) if B > 3 else {}))
    assert ref[0].any()
    print(case[-2], par)


def test_no_carried_membrane():
    r = np.random.Generator(np.random.PCG64(7400))
    s = (r.random((8, 5, 72, 9, 26)) < 0.12).astype(np.uint8)
    w = synth.kaiming_normal(74, 64, 72)
    kw = dict(K=4, beta=0.5, theta=1.0, mode=TP, precision=api.TAC_BF16)
    whole = run_gpu(s, w, **kw)
    assert np.array_equal(run_gpu(s, w, trace=False, **kw)["packed"], whole["packed"])
    # a sample's bits do not depend on the batch
    for b in range(5):
        assert np.array_equal(run_gpu(s[:, b:b + 1], w, trace=False, **kw)["packed"], whole["packed"][:, b:b + 1])
