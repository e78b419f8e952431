"""Which layers the matrix-core kernel of the first layers takes: host rules, compiled into a small library of their own
(first_plan_shim.cpp)."""
import ctypes
import os
import subprocess

import pytest

from paper_2603_13810_amd import api, build
from test_gpu_first import TILES

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("first") / "first_plan.so")
    subprocess.check_call([build.hipcc(), "--offload-arch=gfx950", "-O1", "-std=c++20", "-fPIC", "-shared", "-x", "hip", "-I",
                           build.INCLUDE, "-I", build.CSRC, os.path.join(HERE, "first_plan_shim.cpp"), "-o", lib])
    return ctypes.CDLL(lib)


FIELDS = ("pairs", "blocks", "pair_tiles", "co_tiles", "workgroups", "lds")


@pytest.fixture(scope="module")
def plan(shim):
    def of(desc, trace=False, state=False):
        out = (ctypes.c_longlong * len(FIELDS))()
        shim.first_plan_of(ctypes.byref(desc), int(trace), int(state), out)
        return dict(zip(FIELDS, out))
    return of


def _desc(B, Cin, Cout, H, W, stride=1, precision=api.TAC_FP32, **kw):
    return api.make_desc(1, B, Cin, H, W, Cout, K=1, beta=0.9, theta=1.0, mode=api.TAC_PER_STEP, stride=stride, precision=precision, **kw)


# (Cin, Cout, H, W, stride): planes of 2^28 neurons and more, and the last ones below
@pytest.mark.parametrize("shape,taken", [((1, 5, 2 ** 21, 128, 1), False), ((2, 7, 2 ** 21 + 1, 128, 1), False), ((1, 6, 2 ** 23, 128, 2), False),
                                         ((1, 5, 2 ** 28, 1, 1), False), ((1, 4, 2 ** 22 - 1, 128, 1), True), ((1, 1, 2 ** 23, 128, 1), True),
                                         ((1, 5, 2 ** 21 - 16, 128, 1), True), ((2, 8, 28, 28, 1), True), ((3, 8, 28, 28, 1), False),
                                         ((1, 8, 28, 129, 1), False)])
def test_membranes_of_fp32_layers_are_within_reach(shim, shape, taken):
    Cin, Cout, H, W, stride = shape
    d = _desc(1, Cin, Cout, H, W, stride)
    api.tac_out_shape(d)                                       # an accepted layer
    assert bool(shim.fp32_layer_on_matrix_cores(ctypes.byref(d))) == taken
    if taken and Cin <= 2:
        # the kernel's largest 32-bit membrane offset: four planes for the upper lane half (where it has channels), the tile's 16 rows
        Ho, Wo = (H - 1) // stride + 1, (W - 1) // stride + 1
        assert 4 * (16 * Wo + (4 * Ho * Wo if Cout > 4 else 0)) < 2 ** 32


def test_a_caller_who_asks_for_the_vector_kernel_gets_it(shim):
    for kernel, taken in ((api.TAC_KERNEL_AUTO, True), (api.TAC_KERNEL_DIRECT, False)):
        d = _desc(4, 1, 8, 28, 28, kernel=kernel)
        assert bool(shim.fp32_layer_on_matrix_cores(ctypes.byref(d))) == taken
        assert api.tac_select_kernel(d) == api.TAC_KERNEL_DIRECT and api.tac_prepared_weight_bytes(d) == 9 * 32 * 4    # one layout


# (B, Cout, H, W): launches of 2^32 threads and more, which a grid in one dimension cannot have, and of fewer; more channels than the
# vector kernel has ever taken (its refusal stays)
@pytest.mark.parametrize("shape,taken", [((65535, 8, 2049, 1), False), ((65535, 1, 2049, 15), False), ((65535, 8, 2000, 2), True),
                                         ((1, 32 * 65536, 8, 1), False), ((1, 32 * 65535, 8, 1), True)])
def test_launches_of_fp32_layers_fit_a_grid(shim, shape, taken):
    B, Cout, H, W = shape
    d = _desc(B, 1, Cout, H, W)
    api.tac_out_shape(d)                                       # an accepted layer
    assert bool(shim.fp32_layer_on_matrix_cores(ctypes.byref(d))) == taken


@pytest.mark.parametrize("name", TILES)
def test_case_has_the_tiles_it_is_there_for(plan, name):
    (Cin, Cout, H, W, stride, B, T, K, mode, pooled), (pairs, blocks, rest) = TILES[name]
    for precision in (api.TAC_BF16,) if pooled else (api.TAC_BF16, api.TAC_FP32):
        d = _desc(B, Cin, Cout, H, W, stride, precision, **(dict(out_format=api.TAC_OUT_BITS_MAXPOOL2) if pooled else {}))
        got = plan(d)
        Ho, words = (H - 1) // stride + 1, ((W - 1) // stride + 32) // 32
        in_all = Ho // 2 * words if pooled else (Ho * words + 1) // 2
        assert (got["pairs"], got["blocks"], in_all - got["pairs"] * (got["pair_tiles"] - 1)) == (pairs, blocks, rest)
        assert got["workgroups"] >= 512


def test_lds_of_a_workgroup(plan):
    # more than 64 KiB only where the launch asks for it (up to 80 KiB, two workgroups per compute unit), and the largest case of
    # test_gpu_first.py is there
    largest = 0
    for precision in (api.TAC_FP32, api.TAC_BF16):
        for W in range(1, 129):
            for stride in (1, 2):
                for Cout in (8, 64, 96, 128):
                    for pooled in (False, True):
                        if pooled and (precision == api.TAC_FP32 or W % 2 or (W // stride) % 2):
                            continue
                        d = _desc(512, 2, Cout, 256, W, stride, precision, **(dict(out_format=api.TAC_OUT_BITS_MAXPOOL2) if pooled else {}))
                        for trace in (False, True):
                            largest = max(largest, plan(d, trace, True)["lds"])
    assert largest <= 80 * 1024
    assert plan(_desc(64, 2, 32, 128, 128, 2), state=True) == dict(pairs=8, blocks=1, pair_tiles=8, co_tiles=1, workgroups=512, lds=largest)
