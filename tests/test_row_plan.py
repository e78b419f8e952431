"""Which bf16 layers run on the row kernel, and whether a launch's plan covers the layer: the host rules of tac_row_plan.h, compiled into a library of their
own (row_plan_shim.cpp)."""
import ctypes
import os
import random
import subprocess

import pytest

from paper_2603_13810_amd import api, build
from test_gpu_row import CASES

HERE = os.path.dirname(os.path.abspath(__file__))
FIELDS = ("kp", "pw", "nco", "nnp", "waves", "flatten", "spr", "tr", "lr", "row_tiles", "co_tiles", "cb", "parts", "lrp", "n_jobs", "lds", "nks")


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("plan") / "row_plan.so")
    subprocess.check_call([build.hipcc(), "--offload-arch=gfx950", "-O1", "-std=c++20", "-fPIC", "-shared", "-x", "hip", "-I",
                           build.INCLUDE, "-I", build.CSRC, os.path.join(HERE, "row_plan_shim.cpp"), "-o", lib])
    shim = ctypes.CDLL(lib)

    def of(desc, traced=False):
        out = (ctypes.c_int * len(FIELDS))()
        return dict(zip(FIELDS, out)) if shim.row_plan_of(ctypes.byref(desc), int(traced), 2, out) else None
    return of


def _desc(B, Cin, Cout, H, W, stride, mode, K, T, **kw):
    return api.make_desc(T, B, Cin, H, W, Cout, K=K, beta=0.9, theta=1.0, mode=mode, stride=stride, precision=api.TAC_BF16, **kw)


@pytest.mark.parametrize("case", CASES, ids=[c[-2] for c in CASES])
def test_case_takes_the_variant_it_is_there_for(plan, case):
    B, Cin, Cout, H, W, stride, mode, K, T, _, want = case
    d = _desc(B, Cin, Cout, H, W, stride, mode, K, T)
    assert api.tac_select_kernel(d) == api.TAC_KERNEL_MFMA
    got = plan(d)
    assert {k: got[k] for k in want} == want


def test_plans_cover_their_layers(plan):
    r = random.Random(7)
    taken = 0
    for _ in range(3000):
        stride, mode = r.choice([1, 2]), r.choice([api.TAC_PER_STEP, api.TAC_COLLAPSE, api.TAC_PRESERVE])
        K = 1 if mode == api.TAC_PER_STEP else r.randint(1, 18)
        B, Cin, Cout, H, W, T = r.choice([1, 2, 7, 60, 300]), 8 * r.randint(1, 17), r.randint(1, 260), r.randint(1, 140), r.randint(16, 66) * stride, r.randint(1, 40)
        q = plan(_desc(B, Cin, Cout, H, W, stride, mode, K, T))
        Ho, Wo, K = (H - 1) // stride + 1, (W - 1) // stride + 1, min(K, T)
        if q is None:
            continue
        taken += 1
        assert Cin <= 128 and K <= 16 and 16 < Wo <= 64 and q["kp"] >= K
        assert q["pw"] * q["nco"] <= q["waves"] <= (16 if q["nnp"] == 1 else 12) and q["lds"] <= 160 * 1024
        # rows and channels: every one has a tile, a tile's segments fit its blocks and its LDS rows the image's
        rows = B * Ho if q["flatten"] else Ho
        assert q["row_tiles"] * q["tr"] >= rows > (q["row_tiles"] - 1) * q["tr"]
        assert q["spr"] * 16 >= Wo > (q["spr"] - 1) * 16 and q["tr"] * q["spr"] <= 2 * q["pw"] * q["nnp"]
        assert q["lr"] >= (q["tr"] - 1) * stride + 3 and q["co_tiles"] * 32 * q["nco"] >= Cout and q["nks"] * 16 >= 9 * Cin
        if q["flatten"]:
            most = max(((f + min(q["tr"], rows - f) - 1) // Ho) - f // Ho for f in range(0, rows, q["tr"]))
            assert q["lr"] >= (q["tr"] - 1) * stride + 3 + most * (3 - stride)
        # jobs: every LDS row and channel has one, none is empty, and a job's words are no more than a wave has registers for
        assert q["parts"] * q["lrp"] >= q["lr"] > (q["parts"] - 1) * q["lrp"]
        assert q["n_jobs"] == -(-(Cin // 8) // q["cb"]) * q["parts"]
        assert 8 * q["cb"] * q["lrp"] * ((W + 31) // 32) <= 64 * {1: 8, 2: 8, 4: 6, 8: 4, 16: 2}[q["kp"]]
    assert taken > 1000


def test_forms_that_stay_on_the_older_kernels(plan):
    ok = (24, 48, 80, 45, 45, 1, api.TAC_COLLAPSE, 4, 8)
    assert plan(_desc(*ok)) and not plan(_desc(*ok), traced=True)
    assert plan(_desc(*ok, in_format=api.TAC_IN_BITS_POOL2)) is None and plan(_desc(*ok, in_format=api.TAC_IN_BITS_MAXPOOL2)) is None
    assert plan(_desc(*ok, in_format=api.TAC_IN_F32)) is None and plan(_desc(*ok, out_format=api.TAC_OUT_BITS_MAXPOOL2)) is None
    fp32 = _desc(*ok)
    fp32.precision = api.TAC_FP32
    assert plan(fp32) is None
    assert plan(_desc(24, 44, *ok[2:])) is None and plan(_desc(24, 136, *ok[2:])) is None                # channels
    assert plan(_desc(*ok[:7], 17, 34)) is None                                                          # frames of a group
    assert plan(_desc(24, 48, 80, 45, 16, *ok[5:])) is None and plan(_desc(24, 48, 80, 45, 65, *ok[5:])) is None     # pixels of a row
    assert plan(_desc(8, 8, 120, 16, 24, 1, api.TAC_PRESERVE, 2, 10)) is None                            # too little to do
    assert plan(_desc(4096, 128, 8, 512, 64, 1, api.TAC_COLLAPSE, 16, 16)) is None                       # a group's words: 2^31 bytes and more


def test_lengths_up_to_the_next_power_of_two_groups_share_a_plan(plan):
    # (with a shorter last group a second table takes its place in the LDS)
    r = random.Random(8)
    for _ in range(300):
        K, B, Cin = r.randint(2, 16), r.choice([1, 2, 7, 60]), 8 * r.randint(3, 16)
        rest = (B, Cin, r.randint(8, 200), r.randint(4, 60), r.randint(17, 64), r.choice([1, 2]), api.TAC_COLLAPSE, K)
        plans = [[plan(_desc(*rest, g * K - K + last)) for g in range(17, 33)] for last in (K, 1, K - 1)]
        assert all(p == plans[0][0] for p in plans[0])
        assert all(p == plans[1][0] for p in plans[1] + plans[2])
