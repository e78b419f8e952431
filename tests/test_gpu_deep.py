"""bf16 layers of the direct family on the matrix cores (more than 128 input channels at widths that the large kernel does not take, or rows of aggregates too wide
for the kernel in between): against the oracle, and against the vector kernel, which takes the same prepared weights."""
import numpy as np
import pytest

from paper_2603_13810_amd import api, synth
from gpu_util import check_layer, run_gpu
from parity_util import compare

pytestmark = pytest.mark.gpu
TAC, TP, STEP = api.TAC_COLLAPSE, api.TAC_PRESERVE, api.TAC_PER_STEP

# (B, Cin, Cout, H, W, stride, mode, K, T, what, what the launch's plan has in it: test_deep_plan.py holds the choice to it on the CPU)
CASES = [
    (1, 136, 120, 1, 1, 1, STEP, 1, 27, "one pixel", dict(kp=1, gb=4, rpb=16)),
    (3, 192, 33, 5, 3, 1, TAC, 2, 9, "a last group of one, a tile of one channel, three samples a tile", dict(kp=2, rpb=8, flatten=1)),
    (2, 192, 64, 12, 12, 2, TP, 3, 11, "stride 2, a last group of two", dict(kp=4, rpb=4)),
    (24, 256, 256, 13, 13, 2, STEP, 1, 3, "two blocks a workgroup, a group at a time", dict(kp=1, pb=2, gb=1)),
    (20, 136, 256, 8, 8, 1, TAC, 2, 9, "two blocks a workgroup, two groups at a time", dict(kp=2, pb=2, gb=2)),
    (2, 200, 40, 9, 16, 1, TAC, 4, 20, "rows of 16, five groups", dict(kp=4, rpb=2)),
    (2, 144, 96, 7, 23, 1, TP, 8, 17, "a row a block, two tables", dict(kp=8, rpb=1)),
    (1, 168, 32, 6, 45, 1, TP, 5, 12, "two words a row", dict(kp=8, pb=2)),
    (2, 256, 48, 10, 8, 1, TAC, 16, 33, "groups of 16, one frame left over", dict(kp=16)),
    (1, 192, 130, 8, 31, 2, TP, 12, 26, "groups of 12, stride 2", dict(kp=16)),
    (3, 96, 96, 17, 64, 2, TAC, 8, 17, "few channels, wide rows, stride 2", dict(kp=8, rpb=1)),
    (2, 128, 64, 5, 127, 2, STEP, 1, 5, "rows of 127 pixels", dict(kp=1, pb=2, gb=1)),
]


@pytest.mark.parametrize("case", CASES, ids=[c[-2] for c in CASES])
def test_layer(case):
    B, Cin, Cout, H, W, stride, mode, K, T = case[:9]
    r = np.random.Generator(np.random.PCG64(7100 + Cin + Cout + H + W + K))
    s = (r.random((T, B, Cin, H, W)) < 0.12).astype(np.uint8)
    w = synth.kaiming_normal(71, Cout, Cin) * np.float32(1.5)
    bias = (r.standard_normal(Cout) * 0.1).astype(np.float32)
    Ho, Wo = (H - 1) // stride + 1, (W - 1) // stride + 1
    v0 = (r.standard_normal((B, Cout, Ho, Wo)) * 0.3).astype(np.float32)
    kw = dict(K=K, beta=0.9, theta=1.0, mode=mode, stride=stride, precision=api.TAC_BF16, bias=bias, v0=v0)
    par, g, ref = check_layer(s, w, expect_kernel=api.TAC_KERNEL_DIRECT, **kw, **(dict(oracle_samples=[0, B - 1]) if B > 3 else {}))
    assert ref[0].any()
    # the vector kernel on the same prepared weights: fp32 sums of the same products in another order, K steps of each in TAC-TP
    v = run_gpu(s, w, kernel=api.TAC_KERNEL_DIRECT, **kw)
    both = compare(v["spikes"], v["v_trace"].astype(np.float64), g.get("spikes_all", g["spikes"]), run_gpu(s, w, **kw)["v_trace"], 1.0, 2e-5)
    assert both.ok, both
    print(case[-2], par, both)


def test_no_carried_membrane():
    r = np.random.Generator(np.random.PCG64(7200))
    s = (r.random((8, 5, 160, 9, 10)) < 0.12).astype(np.uint8)
    w = synth.kaiming_normal(72, 64, 160)
    kw = dict(K=2, beta=0.5, theta=1.0, mode=TP, precision=api.TAC_BF16)
    whole = run_gpu(s, w, **kw)
    assert np.array_equal(run_gpu(s, w, trace=False, **kw)["packed"], whole["packed"])
    # a sample's bits do not depend on the batch
    for b in range(5):
        assert np.array_equal(run_gpu(s[:, b:b + 1], w, trace=False, **kw)["packed"], whole["packed"][:, b:b + 1])
