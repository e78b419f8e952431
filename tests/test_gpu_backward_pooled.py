"""The LIF recurrence backwards through the 2 x 2 max pool in the writer: the pooled kernels (one and two windows per
thread, and the scalar form for addresses that are not aligned) against the unpooled recurrence on gradients that the
test routes itself."""
import numpy as np
import pytest
import torch

from paper_2603_13810_amd import api

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _route(v, g, theta):
    """Gradient of the pooled spikes [T,B,C,H/2,W/2] to the first maximal spike of each window: [T,B,C,H,W]."""
    T, B, C, H, W = v.shape
    win = (v >= theta).reshape(T, B, C, H // 2, 2, W // 2, 2).transpose(0, 1, 2, 3, 5, 4, 6).reshape(T, B, C, H // 2, W // 2, 4)
    first = np.where(win.any(-1), win.argmax(-1), 0)
    out = np.zeros(win.shape, np.float32)
    np.put_along_axis(out, first[..., None], g[..., None], -1)
    return out.reshape(T, B, C, H // 2, W // 2, 2, 2).transpose(0, 1, 2, 3, 5, 4, 6).reshape(T, B, C, H, W)


# (B, Cout, H, W, element offset of the membranes): rows of 2, 6 and 8 pixels, both sides of the size at which a thread
# takes two windows, addresses that are 8- and 4-byte aligned only
SHAPES = [(3, 5, 2, 2, 0), (2, 7, 6, 6, 0), (2, 3, 4, 8, 0), (4, 64, 64, 64, 0), (4, 66, 64, 62, 0), (4, 64, 64, 64, 2), (2, 3, 4, 8, 1)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("mode,K,T,Kc", [(api.TAC_PER_STEP, 1, 5, 0), (api.TAC_COLLAPSE, 2, 7, 0), (api.TAC_PRESERVE, 4, 6, 4)])
def test_pooled_recurrence_is_the_unpooled_one_on_routed_gradients(shape, mode, K, T, Kc):
    B, C, H, W, off = shape
    r = np.random.Generator(np.random.PCG64(B + C + H + W + T))
    kw = dict(K=K, beta=0.9, theta=1.0, mode=mode, precision=api.TAC_BF16)
    pooled = api.make_desc(T, B, 8, H, W, C, out_format=api.TAC_OUT_BITS_MAXPOOL2, **kw)
    plain = api.make_desc(T, B, 8, H, W, C, **kw)
    T_out = api.tac_out_shape(plain)[0]
    n = T_out * B * C * H * W
    buf = torch.empty((n + off,), dtype=torch.float32, device=DEV)
    v = (0.6 * r.standard_normal((T_out, B, C, H, W)) + 0.3).astype(np.float32)
    buf[off:].copy_(torch.from_numpy(v.reshape(-1)))
    vt = buf[off:].view(T_out, B, C, H, W)
    steps = -(-T_out // Kc) if Kc else T_out
    g = r.standard_normal((steps, B, C, H // 2, W // 2)).astype(np.float32)
    idx = np.arange(T_out)
    f = np.ones(T_out, np.float32)
    if Kc:
        f = np.array([np.float32(0.5 ** (min(Kc, T_out - n // Kc * Kc) - 1 - n % Kc)) for n in idx], np.float32)
    per_step = f[:, None, None, None, None] * g[idx // Kc if Kc else idx]
    s = torch.zeros((T, B, 8, H, (W + 31) // 32), dtype=torch.int32, device=DEV)
    w = torch.zeros((C, 8, 3, 3), dtype=torch.float32, device=DEV)
    got = api.tac_conv_lif_backward(pooled, s, w, vt, torch.from_numpy(g).to(DEV), want_input_grad=False, grad_out_group_K=Kc,
                                    grad_out_group_beta=0.5)
    ref = api.tac_conv_lif_backward(plain, s, w, torch.from_numpy(v).to(DEV), torch.from_numpy(_route(v, per_step, 1.0)).to(DEV),
                                    want_input_grad=False)
    torch.cuda.synchronize()
    a, b = got["grad_y"].cpu().numpy(), ref["grad_y"].cpu().numpy()
    # the same fp32 expressions, contracted by the compiler where it likes: a few units in the last place per step, and a
    # step hands on at most 1 + theta times its error
    assert np.abs(a - b).max() <= T * 4 * 2.0 ** -24 * np.abs(b).max()
    # dW and dbias start from zero (the frames are silent)
    assert not got["grad_w"].any()
    assert torch.allclose(got["grad_bias"].double(), got["grad_y"].double().sum((0, 1, 3, 4)), rtol=0,
                          atol=1e-5 * float(got["grad_y"].double().abs().sum((0, 1, 3, 4)).max()))
