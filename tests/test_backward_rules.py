"""Which kernels a backward call launches: host rules, compiled into a small library of their own (backward_rules_shim.cpp)."""
import ctypes
import os
import subprocess

import pytest

from paper_2603_13810_amd import api, build
from test_gpu_backward_dgrad import CASES, VECTOR
from test_gpu_backward_wgrad import BITS, FIRST, FIRST_TAKEN, INFINITE, REAL

POOLS = {api.TAC_IN_BITS_POOL2: 1, api.TAC_IN_BITS_MAXPOOL2: 2}
HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("rules") / "backward_rules.so")
    subprocess.check_call([build.hipcc(), "--offload-arch=gfx950", "-O1", "-std=c++20", "-fPIC", "-shared", "-x", "hip", "-I", build.INCLUDE,
                           "-I", build.CSRC, os.path.join(HERE, "backward_rules_shim.cpp"), "-o", lib])
    return ctypes.CDLL(lib)


@pytest.mark.parametrize("neurons,channels,aside", [(512 * 4, 512, False), (1024 * 16, 1024, False), (128 * 2 * 4, 128, False),
                                                    (128 * 16 * 16, 128, True), (64 * 8 * 64, 64, True)])
def test_a_large_weight_gradient_is_not_cleared_by_a_handful_of_threads(rules, neurons, channels, aside):
    # four neurons a thread in the recurrence; dW of channels x channels x 9 floats
    threads, floats = ctypes.c_longlong(neurons // 4), ctypes.c_longlong(9 * channels * channels)
    assert bool(rules.clear_in_recurrence(threads, floats)) == aside


# (groups, B, Cin, Cout, H = W, stride, on the matrix cores): the faster side as measured, 1.2 times and more apart
@pytest.mark.parametrize("case", [(8, 64, 1, 64, 64, 1, False), (8, 64, 4, 64, 64, 1, False), (8, 64, 8, 64, 64, 1, True), (8, 64, 16, 8, 64, 1, True),
                                  (8, 64, 16, 64, 64, 1, True), (12, 128, 1, 64, 28, 1, False), (12, 128, 1, 8, 28, 1, False), (4, 4, 3, 64, 200, 1, False),
                                  (4, 4, 3, 16, 200, 1, False), (2, 64, 1, 64, 28, 1, True), (2, 64, 8, 8, 28, 1, True), (2, 64, 4, 64, 28, 1, True), (2, 64, 8, 64, 28, 1, True), (2, 4, 1, 64, 28, 1, True),
                                  (2, 64, 2, 64, 7, 1, True), (7, 128, 32, 64, 14, 1, True), (4, 16, 128, 64, 8, 1, True), (4, 16, 128, 64, 8, 2, False)])
def test_input_gradient_kernel(rules, case):
    G, B, Cin, Cout, hw, stride, matrix = case
    assert bool(rules.input_gradient_on_matrix_cores(G, B, Cin, Cout, hw, hw, stride, 0, 0)) == matrix


def test_the_vector_kernel_has_its_cases(rules):
    for case in CASES:
        B, Cin, Cout, H, W, fmt, per_group, K, T = case
        frames, pool2 = (0 if per_group else K), (0 if fmt == BITS else POOLS[fmt])
        assert bool(rules.input_gradient_on_matrix_cores((T + K - 1) // K, B, Cin, Cout, H, W, 1, frames, pool2)) == (case not in VECTOR)


def test_the_vector_kernel_stays_within_a_grid(rules):
    for Cin in (1, 4, 5, 262139, 262140, 262141, 1 << 20, 2 ** 31 - 1):
        out = (ctypes.c_uint * 2)()
        rules.vector_kernel_tiles(Cin, out)
        assert out[0] <= 65535 and (out[1] - 1) * out[0] * 4 < Cin <= out[0] * out[1] * 4


# (pairs, Cin, Cout, H, W, whether four waves share the output channels): the faster side as measured, 1.2 times and more apart
@pytest.mark.parametrize("case", [(16, 128, 128, 8, 8, True), (30, 64, 64, 8, 8, True), (24, 10, 32, 9, 44, False), (16, 16, 48, 31, 32, False),
                                  (2, 40, 48, 63, 41, False), (6, 2, 48, 64, 27, False), (64, 128, 16, 8, 8, False), (8, 1, 16, 28, 28, False), (20, 12, 64, 12, 55, False)])
def test_which_input_gradients_share_output_channels(rules, case):
    pairs, Cin, Cout, H, W, splits = case
    assert bool(rules.input_gradient_splits(1, pairs, Cin, Cout, H, W, 0, 0)) == splits


# Values for each frame of a group: (groups, B, Cin, Cout, H, W, K, pool on load (0 none, 1 mean, 2 max), shared): the faster side as measured, 1.1 times and more apart
@pytest.mark.parametrize("case", [(1, 3, 64, 16, 6, 6, 8, 2, True), (2, 74, 32, 9, 5, 8, 16, 1, True), (1, 4, 40, 40, 34, 10, 8, 1, True), (1, 46, 24, 48, 13, 13, 3, 1, True),
                                  (4, 17, 40, 15, 9, 9, 16, 0, True), (7, 100, 7, 13, 4, 4, 2, 1, False), (1, 3, 35, 2, 36, 36, 3, 0, False),
                                  (1, 112, 1, 6, 27, 3, 4, 2, False), (4, 27, 16, 8, 8, 4, 1, 0, False)])
def test_values_of_every_frame_are_stored_by_more_workgroups(rules, case):
    G, B, Cin, Cout, H, W, K, pool2, splits = case
    assert bool(rules.input_gradient_splits(G, B, Cin, Cout, H, W, K, pool2)) == splits


PLAN = ("ncg", "co_groups", "split", "n_pairs", "rows", "n_strips", "pair_tiles", "lds")


def _first(rules, B, Cin, Cout, H, W, stride, fmt, K, T):
    d = api.make_desc(T, B, Cin, H, W, Cout, K=K, beta=0.9, theta=1.0, mode=api.TAC_COLLAPSE, stride=stride, in_format=fmt)
    out = (ctypes.c_int * len(PLAN))()
    return dict(zip(PLAN, out)) if rules.first_weight_gradient(ctypes.byref(d), out) else None


def test_first_layers_take_the_kernel_they_are_there_for(rules):
    assert [_first(rules, *case) is not None for case in FIRST] == FIRST_TAKEN
    B, Cin, Cout, H, W = INFINITE
    assert _first(rules, B, Cin, Cout, H, W, 1, REAL, 1, 1) and W % 4


# two input channels, bits, few workgroups of one item each: the frames of a group and the turns of the threads that build its aggregates
@pytest.mark.parametrize("case,taken", [((3, 2, 117, 55, 68, 2, BITS, 16, 19), False), ((2, 2, 20, 67, 66, 2, BITS, 8, 15), False), ((2, 2, 118, 48, 66, 2, BITS, 8, 9), False),
                                        ((2, 2, 101, 46, 50, 2, BITS, 4, 4), True), ((3, 1, 117, 55, 68, 2, BITS, 16, 19), True),
                                        ((8, 2, 117, 55, 68, 2, BITS, 16, 19), True), ((16, 2, 52, 51, 57, 2, BITS, 16, 16), True)])
def test_small_first_layers(rules, case, taken):
    assert (_first(rules, *case) is not None) == taken
