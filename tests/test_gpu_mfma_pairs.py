"""The large matrix-core kernel with two groups of frames in hand (grids of at most one workgroup per compute unit): every tile height,
odd and even numbers of groups, ragged rows, pooled output, recorded and carried membranes; and no bit that depends on the tile."""
import numpy as np
import pytest

from paper_2603_13810_amd import api, synth
from gpu_util import check_layer, run_gpu

pytestmark = pytest.mark.gpu

UNITS = 256                     # compute units


def _batch(Ho, Wo, Cout, pixels):
    """A batch whose grid of 64-channel tiles of `pixels` pixels the chip takes in one go, and that of half as high tiles not."""
    tiles = lambda px: -(-Ho // (px // Wo)) * (Cout // 64)
    B = UNITS // tiles(pixels)
    assert B >= 1 and (pixels == 64 or Wo * 2 > pixels or B * tiles(pixels // 2) > UNITS)
    return B


# (input width, stride, input rows, pixels per tile)
TILES = [(32, 1, 11, 64), (32, 1, 11, 128), (32, 1, 19, 256), (32, 2, 13, 64), (32, 2, 35, 128), (32, 2, 67, 256),
         (64, 2, 9, 64), (64, 2, 21, 128), (64, 2, 37, 256), (64, 1, 5, 128), (64, 1, 10, 256)]
# (three groups on tiles of 256 pixels go one at a time, but with recorded membranes)
GROUPS = [(api.TAC_PER_STEP, 1, 3), (api.TAC_COLLAPSE, 2, 4), (api.TAC_PRESERVE, 2, 6), (api.TAC_PRESERVE, 4, 12), (api.TAC_PRESERVE, 2, 10)]


@pytest.mark.parametrize("W,stride,H,pixels", TILES)
@pytest.mark.parametrize("mode,K,T", GROUPS)
def test_pairs_of_groups(W, stride, H, pixels, mode, K, T):
    Ho, Wo = (H - 1) // stride + 1, W // stride
    B = 2 if pixels == 64 else _batch(Ho, Wo, 128, pixels)
    r = np.random.Generator(np.random.PCG64(W + stride + H + K))
    s = (r.random((T, B, 32, H, W)) < 0.15).astype(np.uint8)
    w = synth.kaiming_normal(31, 128, 32)
    bias = (r.standard_normal(128) * 0.1).astype(np.float32)
    v0 = (r.standard_normal((B, 128, Ho, Wo)) * 0.3).astype(np.float32)
    _, g, _ = check_layer(s, w, K=K, beta=0.9, theta=1.0, mode=mode, stride=stride, precision=api.TAC_BF16, bias=bias, v0=v0,
                          expect_kernel=api.TAC_KERNEL_MFMA, oracle_samples=[0, B - 1])
    # one sample alone runs on other tiles (the lowest ones): the same bits
    one = run_gpu(s[:, B - 1:], w, K=K, beta=0.9, theta=1.0, mode=mode, stride=stride, precision=api.TAC_BF16, bias=bias, v0=v0[B - 1:])
    assert np.array_equal(one["packed"], g["packed"][:, B - 1:]) and np.array_equal(one["v_trace"], g["v_trace"][:, -1:])


@pytest.mark.parametrize("W,H,B", [(32, 14, 3), (32, 6, 60), (64, 6, 5), (64, 6, 60)])
@pytest.mark.parametrize("mode,K,T", [(api.TAC_PRESERVE, 4, 12), (api.TAC_COLLAPSE, 2, 8)])
def test_pairs_of_groups_pooled(W, H, B, mode, K, T):
    r = np.random.Generator(np.random.PCG64(W + H + B))
    s = (r.random((T, B, 16, H, W)) < 0.2).astype(np.uint8)
    w = synth.kaiming_normal(32, 128, 16)
    check_layer(s, w, K=K, beta=0.9, theta=1.0, mode=mode, precision=api.TAC_BF16, out_pool=True, expect_kernel=api.TAC_KERNEL_MFMA,
                oracle_samples=[0, B - 1])


@pytest.mark.parametrize("K,T", [(8, 24), (16, 32), (5, 15), (3, 10)])
def test_pairs_of_groups_larger_groups(K, T):
    # K = 3 at T = 10: the shorter last group is a launch of its own behind three whole ones
    r = np.random.Generator(np.random.PCG64(K))
    s = (r.random((T, 2, 48, 11, 32)) < 0.1).astype(np.uint8)
    w = synth.kaiming_normal(33, 256, 48)
    check_layer(s, w, K=K, beta=0.9, theta=1.0, mode=api.TAC_PRESERVE, precision=api.TAC_BF16, expect_kernel=api.TAC_KERNEL_MFMA)
