"""First layers on the matrix cores (1 or 2 input channels, bf16 and fp32): the edges of their tiles against the oracle.  A tile is some
pairs of packed words x some blocks of 32 output channels, chosen by the number of words, channels and samples; groups ask for up to
8 frames together (4 with two input channels); with rows of 65 to 96 pixels a tile starts in the middle of a row."""
import numpy as np
import pytest

from paper_2603_13810_amd import api, synth

from gpu_util import check_layer, run_oracle
from parity_util import TOL_FP32, compare, np_unpack

pytestmark = pytest.mark.gpu
B16, F32 = api.TAC_BF16, api.TAC_FP32
STEP, TAC, TP = api.TAC_PER_STEP, api.TAC_COLLAPSE, api.TAC_PRESERVE

# (Cin, Cout, H, W, stride, B, T, K, mode, what)
CASES = [
    (1, 8, 28, 28, 1, 4, 4, 2, TAC, "one wave per workgroup"),
    (1, 32, 1, 1, 1, 1, 3, 2, TP, "one pixel, a shorter last group"),
    (2, 33, 7, 33, 1, 2, 9, 4, TAC, "a second word of one pixel, a second block of one channel"),
    (2, 96, 9, 90, 1, 2, 6, 3, TP, "three words a row, three blocks"),
    (1, 160, 5, 65, 1, 3, 8, 8, TAC, "three words a row, five blocks in two tiles, eight frames together"),
    (2, 128, 6, 128, 1, 1, 10, 5, TP, "four words a row, four blocks, five frames in two batches"),
    (2, 16, 70, 128, 2, 2, 11, 4, TAC, "more words than threads, stride 2"),
    (1, 40, 33, 63, 2, 2, 25, 16, TAC, "two batches, a shorter last group of nine"),
    (2, 64, 20, 31, 1, 40, 4, 1, STEP, "single frames, many samples"),
    (1, 32, 28, 28, 1, 128, 8, 4, TAC, "tiles of an even number of words that do not divide the sample"),
    (2, 12, 3, 2, 2, 5, 7, 32, TP, "a group longer than the sequence"),
]


@pytest.mark.parametrize("dense", [False, True], ids=["bits", "values"])
@pytest.mark.parametrize("precision", [B16, F32], ids=["bf16", "fp32"])
@pytest.mark.parametrize("case", CASES, ids=[c[-1] for c in CASES])
def test_tiles_of_first_layers(case, precision, dense):
    Cin, Cout, H, W, stride, B, T, K, mode, _ = case
    if dense and precision == F32 and B > 8:
        B = 8
    r = np.random.Generator(np.random.PCG64(9100 + 7 * Cin + Cout + H + W + T + K))
    s = (r.random((T, B, Cin, H, W)) < 0.3).astype(np.uint8)
    if dense:
        s = (s * r.random(s.shape)).astype(np.float32)
    w = synth.kaiming_normal(61, Cout, Cin) * np.float32(1.5)
    bias = (r.standard_normal(Cout) * 0.1).astype(np.float32)
    Ho, Wo = (H - 1) // stride + 1, (W - 1) // stride + 1
    v0 = (r.standard_normal((B, Cout, Ho, Wo)) * 0.3).astype(np.float32)
    par, g, ref = check_layer(s, w, K=K, beta=0.9, theta=1.0, mode=mode, stride=stride, precision=precision, bias=bias, v0=v0,
                              expect_kernel=api.TAC_KERNEL_MFMA if precision == B16 else api.TAC_KERNEL_DIRECT,
                              oracle_samples=None if B <= 8 else [0, B // 2, B - 1])
    assert H * W == 1 or ref[0].sum() > 0
    print("first layer", par)


# Layers of so many samples that a tile has several block pairs: (Cin, Cout, H, W, stride, B, T, K, mode, pool in the writer), and
# (pairs, blocks of 32 channels, pairs of the sample's last tile).  test_first_plan.py holds the choice to them on the CPU.
TILES = {
    "two pairs of four channel blocks, pooled": ((2, 128, 64, 64, 1, 16, 5, 4, TP, True), (2, 4, 2)),
    "eight pairs, three words a row, pooled, a short last tile": ((1, 32, 10, 90, 1, 256, 3, 2, TAC, True), (8, 1, 7)),
    "four pairs, two words a row, pooled, a short last tile": ((2, 64, 14, 34, 1, 128, 4, 3, TP, True), (4, 2, 2)),
    "eight pairs, stride 2, four words a row": ((2, 32, 128, 128, 2, 64, 3, 2, TAC, False), (8, 1, 8)),
    "six pairs, three words a row, a short last tile": ((1, 24, 11, 70, 1, 256, 4, 4, TAC, False), (6, 1, 5)),
    "two pairs of three channel blocks, a last tile of one": ((2, 96, 7, 33, 1, 128, 5, 2, TP, False), (2, 3, 1)),
    "three pairs of two channel blocks, stride 2": ((1, 40, 11, 40, 2, 512, 3, 1, STEP, False), (3, 2, 3)),
    "eight pairs, one word a row": ((2, 9, 32, 17, 1, 400, 4, 3, TAC, False), (8, 1, 8)),
}


# (fp32 first layers have no pool in the writer)
@pytest.mark.parametrize("dense", [False, True], ids=["bits", "values"])
@pytest.mark.parametrize("name,precision", [(n, p) for n in TILES for p in (B16, F32) if p == B16 or not TILES[n][0][-1]])
def test_tiles_of_several_pairs(name, precision, dense):
    Cin, Cout, H, W, stride, B, T, K, mode, pooled = TILES[name][0]
    r = np.random.Generator(np.random.PCG64(9500 + 7 * Cin + Cout + H + W + T + K))
    s = (r.random((T, B, Cin, H, W), dtype=np.float32) < 0.3).astype(np.uint8)
    if dense:
        s = s * r.random(s.shape, dtype=np.float32)
    w = synth.kaiming_normal(69, Cout, Cin) * np.float32(1.5)
    bias = (r.standard_normal(Cout) * 0.1).astype(np.float32)
    Ho, Wo = (H - 1) // stride + 1, (W - 1) // stride + 1
    v0 = r.standard_normal((B, Cout, Ho, Wo), dtype=np.float32) * np.float32(0.3)
    par, g, ref = check_layer(s, w, K=K, beta=0.9, theta=1.0, mode=mode, stride=stride, precision=precision, bias=bias, v0=v0,
                              oracle_samples=[0, 1, B // 2, B - 1], **(dict(out_pool=True) if pooled else {}))
    assert ref[0].any()
    print(name, par)


@pytest.mark.parametrize("Cout", [1, 7, 8, 9, 16, 17])
@pytest.mark.parametrize("Cin,K,T,mode", [(1, 2, 5, TP), (2, 8, 17, TAC), (1, 16, 16, TAC), (2, 1, 3, STEP)])
def test_recorded_membranes_of_few_channels_fp32(Cin, K, T, mode, Cout):
    """Up to 8 and up to 16 channels have kernels that record a quarter and a half of the registers."""
    r = np.random.Generator(np.random.PCG64(9150 + Cin + Cout + K))
    s = (r.random((T, 3, Cin, 13, 37)) < 0.3).astype(np.uint8)
    w = synth.kaiming_normal(68, Cout, Cin) * np.float32(1.5)
    bias = (r.standard_normal(Cout) * 0.1).astype(np.float32)
    v0 = (r.standard_normal((3, Cout, 13, 37)) * 0.3).astype(np.float32)
    for x in (s, (s * r.random(s.shape)).astype(np.float32)):
        par, g, ref = check_layer(x, w, K=K, beta=0.9, theta=1.0, mode=mode, precision=F32, bias=bias, v0=v0)
        print("first layer", par)


@pytest.mark.parametrize("precision", [B16, F32], ids=["bf16", "fp32"])
@pytest.mark.parametrize("Cin", [1, 2])
def test_values_beyond_a_window_do_not_reach_it(Cin, precision):
    """Infinite input values: the outputs whose windows hold none are what they are without (no slot of another pixel, and no frame
    beyond a shorter last group, is multiplied by zero)."""
    T, H, W = 3, 8, 70
    r = np.random.Generator(np.random.PCG64(9200 + Cin))
    x = (r.random((T, 1, Cin, H, W)) * (r.random((T, 1, Cin, H, W)) < 0.3)).astype(np.float32)
    w = synth.kaiming_normal(62, 40, Cin)
    kw = dict(K=2, beta=0.9, theta=1.0, mode=api.TAC_PRESERVE, precision=precision)
    from gpu_util import run_gpu
    clean = run_gpu(x, w, **kw)
    bad = x.copy()
    bad[:, 0, :, 3, 31] = np.inf
    dirty = run_gpu(bad, w, **kw)
    clear = np.ones((H, W), bool)
    clear[2:5, 30:33] = False
    assert np.array_equal(clean["v_trace"][..., clear], dirty["v_trace"][..., clear])
    assert np.array_equal(clean["spikes"][..., clear], dirty["spikes"][..., clear])
    assert not np.isfinite(dirty["v_trace"][..., ~clear]).all()


@pytest.mark.parametrize("case", [CASES[i] for i in (0, 2, 7, 10)], ids=[CASES[i][-1] for i in (0, 2, 7, 10)])
def test_the_vector_kernel_takes_the_same_layers_and_weights(case):
    """fp32 first layers on the kernel that TAC_KERNEL_DIRECT asks for; weights prepared for it serve the automatic choice too."""
    import torch
    Cin, Cout, H, W, stride, B, T, K, mode, _ = case
    r = np.random.Generator(np.random.PCG64(9400 + Cin + Cout + H + W))
    s = (r.random((T, B, Cin, H, W)) < 0.3).astype(np.uint8)
    w = synth.kaiming_normal(67, Cout, Cin) * np.float32(1.5)
    Ho, Wo = (H - 1) // stride + 1, (W - 1) // stride + 1
    kw = dict(K=K, beta=0.9, theta=1.0, mode=mode, stride=stride, precision=F32, v0=(r.standard_normal((B, Cout, Ho, Wo)) * 0.3).astype(np.float32))
    for kernel in (api.TAC_KERNEL_DIRECT, api.TAC_KERNEL_AUTO):
        par, g, ref = check_layer(s, w, kernel=kernel, expect_kernel=api.TAC_KERNEL_DIRECT, **kw)
        print("first layer", par)
    wp = [api.tac_prepare_weights(api.make_desc(T, B, Cin, H, W, Cout, K=K, beta=0.9, theta=1.0, mode=mode, stride=stride, kernel=kernel),
                                  torch.from_numpy(w).cuda()) for kernel in (api.TAC_KERNEL_DIRECT, api.TAC_KERNEL_AUTO)]
    assert torch.equal(*wp)


def test_workgroups_of_more_than_64_kib_of_lds():
    # fp32, two channels of two aggregate tiles of 19 rows of 128 pixels, eight waves that turn their membranes
    r = np.random.Generator(np.random.PCG64(9300))
    s = (r.random((5, 64, 2, 128, 128)) < 0.2).astype(np.uint8)
    w = synth.kaiming_normal(66, 32, 2) * np.float32(1.5)
    v0 = (r.standard_normal((64, 32, 64, 64)) * 0.3).astype(np.float32)
    par, g, ref = check_layer(s, w, K=2, beta=0.9, theta=1.0, mode=TP, stride=2, precision=F32, v0=v0, oracle_samples=[0, 31, 63])
    assert ref[0].any()
    print("first layer", par)


def test_membranes_behind_four_gib_fp32():
    """Six channels of a plane of 2^28 neurons: the first and the last rows against the oracle on those rows alone."""
    import torch
    Cin, Cout, H, W, rows = 1, 6, 2 ** 21 + 3, 128, 10
    dev = torch.device("cuda:0")
    d = api.make_desc(1, 1, Cin, H, W, Cout, K=1, beta=0.9, theta=1.0, mode=STEP, precision=F32)
    g = torch.Generator(device=dev)
    g.manual_seed(93)
    s = (torch.rand((1, 1, Cin, H, W), generator=g, device=dev) < 0.3).to(torch.uint8)
    w = synth.kaiming_normal(65, Cout, Cin) * np.float32(1.5)
    v0 = torch.randn((1, Cout, H, W), generator=g, device=dev) * 0.3
    v, vt = v0.clone(), torch.full((1, 1, Cout, H, W), float("nan"), device=dev)
    out = torch.full((1, 1, Cout, H, W // 32), -1, dtype=torch.int32, device=dev)
    api.tac_conv_lif(d, api.tac_pack_spikes(s), api.tac_prepare_weights(d, torch.from_numpy(w).to(dev)), None, v, out, vt)
    assert not torch.isnan(vt).any()
    for part, inner in ((slice(0, rows), slice(0, rows - 1)), (slice(H - rows, H), slice(1, rows))):     # (a crop's cut row sees padding)
        host = lambda t: np.ascontiguousarray(t[..., part, :].cpu().numpy())
        ref = run_oracle(host(s), w, K=1, beta=0.9, theta=1.0, mode=STEP, v0=host(v0))
        spikes, trace, final = (np.ascontiguousarray(a[..., inner, :]) for a in (np_unpack(host(out), W), host(vt), host(v)))
        par = compare(ref[0][..., inner, :], ref[1][..., inner, :], spikes, trace, 1.0, TOL_FP32)
        assert par.ok and par.flips == 0, par
        assert np.abs(final - ref[2][..., inner, :]).max() <= 1e-5 * max(1.0, np.abs(ref[2]).max())
