"""Which bf16 layers of the direct family run on the matrix cores, and whether a launch's plan covers the layer: the host rules of
tac_deep_plan.h, compiled into a library of their own (deep_plan_shim.cpp)."""
import ctypes
import os
import random
import subprocess

import pytest

from paper_2603_13810_amd import api, build
from test_gpu_deep import CASES

HERE = os.path.dirname(os.path.abspath(__file__))
FIELDS = ("kp", "pb", "gb", "flatten", "rpb", "tr", "lr", "row_tiles", "co_tiles", "nseg", "xs", "lds", "group")


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("plan") / "deep_plan.so")
    subprocess.check_call([build.hipcc(), "--offload-arch=gfx950", "-O1", "-std=c++20", "-fPIC", "-shared", "-x", "hip", "-I",
                           build.INCLUDE, "-I", build.CSRC, os.path.join(HERE, "deep_plan_shim.cpp"), "-o", lib])
    shim = ctypes.CDLL(lib)

    def of(desc):
        out = (ctypes.c_int * len(FIELDS))()
        return dict(zip(FIELDS, out)) if shim.deep_plan_of(ctypes.byref(desc), out) else None
    shim.deep_loads_outside.restype = ctypes.c_longlong
    of.loads_outside = lambda desc: shim.deep_loads_outside(ctypes.byref(desc))
    return of


def _desc(B, Cin, Cout, H, W, stride, mode, K, T, **kw):
    return api.make_desc(T, B, Cin, H, W, Cout, K=K, beta=0.9, theta=1.0, mode=mode, stride=stride, precision=api.TAC_BF16, **kw)


@pytest.mark.parametrize("case", CASES, ids=[c[-2] for c in CASES])
def test_case_takes_the_variant_it_is_there_for(plan, case):
    B, Cin, Cout, H, W, stride, mode, K, T, _, want = case
    d = _desc(B, Cin, Cout, H, W, stride, mode, K, T)
    assert api.tac_select_kernel(d) == api.TAC_KERNEL_DIRECT
    got = plan(d)
    assert {k: got[k] for k in want} == want


def test_plans_cover_their_layers(plan):
    r = random.Random(5)
    taken = 0
    for _ in range(4000):
        stride, mode = r.choice([1, 2]), r.choice([api.TAC_PER_STEP, api.TAC_COLLAPSE, api.TAC_PRESERVE])
        K = 1 if mode == api.TAC_PER_STEP else r.randint(1, 20)
        B, Cin, Cout, H, W, T = r.choice([1, 2, 7, 300]), 8 * r.randint(1, 36), r.randint(1, 300), r.randint(1, 140), r.randint(1, 140), r.randint(1, 40)
        d = _desc(B, Cin, Cout, H, W, stride, mode, K, T)
        q = plan(d)
        Ho, Wo, K = (H - 1) // stride + 1, (W - 1) // stride + 1, min(K, T)
        if q is None:
            continue
        taken += 1
        assert 16 <= Cin <= 256 and K <= 16 and Wo <= 64 and q["kp"] >= K and q["gb"] * q["pb"] <= 4
        assert q["lds"] <= 160 * 1024 and q["gb"] * q["group"] <= q["lds"]
        # rows: every output row has a tile, a tile's rows fit its blocks, its LDS rows the image's
        rows = B * Ho if q["flatten"] else Ho
        assert q["row_tiles"] * q["tr"] >= rows > (q["row_tiles"] - 1) * q["tr"]
        assert q["tr"] <= q["pb"] // ((Wo + 31) // 32) * q["rpb"] and q["lr"] >= (q["tr"] - 1) * stride + 3
        assert q["rpb"] * min(32, 1 << (Wo - 1).bit_length()) <= 32 or q["rpb"] == 1
        assert q["nseg"] * q["xs"] >= W > (q["nseg"] - 1) * q["xs"] and q["xs"] in (8, 16, 32)
        assert q["co_tiles"] * 32 >= Cout
    assert taken > 500


def test_frame_loads_stay_inside_the_descriptor(plan):
    # a shorter last group that is alone in its round: its round has fewer frames than the others
    assert plan.loads_outside(_desc(3, 192, 33, 5, 3, 1, api.TAC_COLLAPSE, 2, 9)) == 0
    assert plan.loads_outside(_desc(2, 256, 48, 10, 8, 1, api.TAC_COLLAPSE, 16, 33)) == 0
    r = random.Random(6)
    taken = 0
    for _ in range(2000):
        K, B, Cin = r.randint(1, 16), r.choice([1, 2, 7]), 8 * r.randint(2, 32)
        d = _desc(B, Cin, r.randint(1, 80), r.randint(1, 40), r.randint(1, 70), r.choice([1, 2]), api.TAC_COLLAPSE, K, r.randint(1, 40))
        outside = plan.loads_outside(d)
        taken += outside >= 0
        assert outside <= 0
    assert taken > 500


def test_forms_that_stay_on_the_vector_kernel(plan):
    ok = (2, 192, 64, 12, 12, 2, api.TAC_COLLAPSE, 2, 8)
    assert plan(_desc(*ok))
    assert plan(_desc(*ok, in_format=api.TAC_IN_BITS_POOL2)) is None and plan(_desc(*ok, in_format=api.TAC_IN_BITS_MAXPOOL2)) is None
    assert plan(_desc(*ok, in_format=api.TAC_IN_F32)) is None
    fp32 = _desc(*ok)
    fp32.precision = api.TAC_FP32
    assert plan(fp32) is None
    assert plan(_desc(2, 196, *ok[2:])) is None and plan(_desc(2, 264, *ok[2:])) is None                # channels
    assert plan(_desc(*ok[:7], 17, 34)) is None                                                          # frames of a group
    assert plan(_desc(2, 192, 64, 4, 130, 2, api.TAC_COLLAPSE, 2, 8)) is None                            # rows of 65 pixels
    assert plan(_desc(1, 256, 8, 4, 128, 2, api.TAC_COLLAPSE, 2, 8)) is None                             # three rows of aggregates fill more than the LDS
    assert plan(_desc(1, 192, 6, 16384, 32768 // 64, 1, api.TAC_COLLAPSE, 2, 8)) is None                 # W = 512
