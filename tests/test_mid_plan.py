"""Which tile the in-between matrix-core kernel takes for a layer: the cases of test_gpu_mid.py that are there for a variant
of the kernel take it, and no layer it accepts is left without a tile.  The choice is host code: it is compiled into a
small library of its own (mid_plan_shim.cpp)."""
import ctypes
import os
import random
import subprocess
import time

import pytest

from paper_2603_13810_amd import api, build
import test_gpu_mid_split
from test_gpu_mid import VARIANTS

HERE = os.path.dirname(os.path.abspath(__file__))
FIELDS = ("kp", "nmc", "nnp", "direct", "jobs", "loaders", "batches", "flatten", "rpb", "workgroups", "lds", "split", "nco")


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("plan") / "mid_plan.so")
    subprocess.check_call([build.hipcc(), "--offload-arch=gfx950", "-O1", "-std=c++20", "-fPIC", "-shared", "-x", "hip", "-I",
                           build.INCLUDE, "-I", build.CSRC, os.path.join(HERE, "mid_plan_shim.cpp"), "-o", lib])
    return ctypes.CDLL(lib)


@pytest.fixture(scope="module")
def plan(shim):
    def of(B, Cin, Cout, H, W, stride, pool, out_pool, precision, mode, K, T, trace=False):
        desc = api.make_desc(T, B, Cin, H, W, Cout, K=K, beta=0.9, theta=1.0, mode=mode, stride=stride, precision=precision,
                             in_format={False: api.TAC_IN_BITS, True: api.TAC_IN_BITS_POOL2, "max": api.TAC_IN_BITS_MAXPOOL2}[pool],
                             out_format=api.TAC_OUT_BITS_MAXPOOL2 if out_pool else api.TAC_OUT_BITS)
        out = (ctypes.c_int * len(FIELDS))()
        rc = shim.mid_plan_of(ctypes.byref(desc), int(trace), out)
        return dict(zip(FIELDS, out)) if rc == 1 else rc
    return of


@pytest.mark.parametrize("name", VARIANTS)
def test_case_takes_the_variant_it_is_there_for(plan, name):
    case, plain = VARIANTS[name][:2]
    with_trace = VARIANTS[name][2] if len(VARIANTS[name]) > 2 else plain
    for want, got in ((plain, plan(*case)), (with_trace, plan(*case, trace=True))):
        assert {k: got[k] for k in want} == want
    if "two pixels a thread" in name:
        assert case[1] // 8 * 4 * case[4] > 256                # at least four rows of aggregates


@pytest.mark.parametrize("name", test_gpu_mid_split.VARIANTS)
def test_case_of_shared_blocks_and_tiles_takes_its_variant(plan, name):
    case, want = test_gpu_mid_split.VARIANTS[name]
    for trace in (False, True):
        got = plan(*case, trace=trace)
        assert {k: got[k] for k in want} == want
        if "two samples" in name:
            assert ((case[3] - 1) // case[5] + 1) % got["rpb"] != 0


@pytest.mark.parametrize("case", test_gpu_mid_split.CASES, ids=[c[-1] for c in test_gpu_mid_split.CASES])
def test_cases_of_waves_that_share_a_block(plan, case):
    B, Cin, Cout, H, W, stride, out_pool, mode, K, T, what = case
    for trace in (False, True):
        got = plan(B, Cin, Cout, H, W, stride, False, out_pool, api.TAC_BF16, mode, K, T, trace)
        assert got["split"] == (4 if "four waves" in what else 8)


def test_batches_on_either_side_of_the_rule(plan):
    for batches, shared in ((test_gpu_mid_split.SHARED, True), (test_gpu_mid_split.ALONE, False)):
        for B in batches:
            got = plan(B, 128, 128, 16, 16, 1, False, False, api.TAC_BF16, api.TAC_PRESERVE, 4, 8, True)
            assert bool(got["split"]) == shared


def test_single_frames_of_few_channels_share_the_compute_units(plan):
    # one workgroup of two pixel blocks per compute unit, 251 of them, takes 52 us a call; twice as many smaller ones without
    # staging 33 us
    got = plan(17, 8, 32, 59, 39, 1, False, False, api.TAC_BF16, api.TAC_PER_STEP, 1, 18)
    assert got["direct"] == 1 and got["nnp"] == 1 and got["workgroups"] >= 2 * 251


def test_every_layer_it_accepts_has_a_tile(plan):
    r = random.Random(3)
    seen = 0
    for _ in range(4000):
        stride, K = r.choice([1, 2]), r.choice([1, 2, 3, 4, 7, 8, 15, 16, 24, 32])
        got = plan(r.choice([1, 3, 20]), 8 * r.randint(1, 16), r.choice([5, 32, 64, 130]), r.choice([1, 2, 9, 30]), r.randint(1, 128), stride,
                   r.choice([False, True, "max"]), False, r.choice([api.TAC_FP32, api.TAC_BF16]), api.TAC_COLLAPSE, K, K, r.random() < 0.5)
        assert got != -1
        if got:
            seen += 1
            assert got["lds"] <= 160 * 1024 and got["loaders"] in (1, 2, 4)
    assert seen > 1500


def test_layers_of_a_network_do_not_turn_each_others_tiles_out(shim):
    # the choice takes up to 18 us, a launch that remembers it a fraction of one: a pass over sixteen layers remembers them all
    descs = [api.make_desc(16, 16, 128, hw, hw, 128, K=K, beta=0.9, theta=1.0, mode=mode, precision=api.TAC_BF16)
             for hw in (4, 8, 12, 16) for K in (2, 4) for mode in (api.TAC_COLLAPSE, api.TAC_PRESERVE)]

    def us(layers):
        best = 1e9
        for _ in range(5):
            t = time.perf_counter()
            for _ in range(50):
                for d in layers:
                    assert shim.mid_launch_of(ctypes.byref(d)) == 0
            best = min(best, (time.perf_counter() - t) / 50 / len(layers) * 1e6)
        return best
    alone = max(us([d]) for d in descs)
    assert us(descs) < 2 * alone + 0.5
