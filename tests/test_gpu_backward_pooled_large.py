"""The LIF recurrence behind a pooled output where its membranes are read past the caches (256 MiB and more): the same dL/dY as the samples give
in calls of a few, which read them through the caches."""
import pytest
import torch

from paper_2603_13810_amd import api

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# (B, Cout, H, W, K, T, frames per group of the layer behind)
@pytest.mark.parametrize("case", [(18, 64, 64, 64, 4, 17, 4), (40, 24, 62, 68, 1, 17, 0), (9, 128, 66, 60, 1, 16, 3)])
def test_membranes_read_once(case):
    B, C, H, W, K, T, Kn = case
    r = torch.Generator(device=DEV)
    r.manual_seed(8100 + C + H)
    mode = api.TAC_PRESERVE if K > 1 else api.TAC_PER_STEP

    def back(first, last):
        desc = api.make_desc(T, last - first, 2, H, W, C, K=K, beta=0.9, theta=1.0, mode=mode, out_format=api.TAC_OUT_BITS_MAXPOOL2)
        return api.tac_conv_lif_backward(desc, x[:, first:last].contiguous(), w, v[:, first:last].contiguous(), g[:, first:last].contiguous(),
                                         want_input_grad=False, grad_out_group_K=Kn, grad_out_group_beta=0.9 if Kn else 0.0)["grad_y"]
    x = torch.zeros((T, B, 2, H, (W + 31) // 32), dtype=torch.int32, device=DEV)
    w = torch.zeros((C, 2, 3, 3), device=DEV)
    v = 0.6 * torch.randn((T, B, C, H, W), generator=r, device=DEV) + 0.7
    g = torch.randn((-(-T // Kn) if Kn else T, B, C, H // 2, W // 2), generator=r, device=DEV)
    assert v.numel() >= 64 << 20
    got = back(0, B)
    for first in range(0, B, 6):
        part = back(first, min(B, first + 6))
        # the same fp32 operations, up to what the compiler fuses
        assert torch.allclose(got[:, first:first + 6], part, rtol=1e-5, atol=1e-6)
