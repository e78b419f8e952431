"""The calls a user of this library makes, as cases that can be timed and compared.

A case is a dict of plain values.  `kind` says what one pass is:

  layer     one tac_conv_lif call, the membrane carried in and out (streaming use)
  frames    raw 0/1 frames (bytes) are packed, then run through a first layer
  stack     a whole network forward, tac_stack_forward; `readout` unpacks its last spikes for a head that follows
  train     a training step without the optimiser: weights prepared again (they change every step), forward with
            the membranes recorded, backward through the stack
  blocks    the blocks of a network one by one, each on spikes of its own: in a deep network one spike that flips in
            its last bit reaches everything behind it, so deep ones are compared block by block
  blocks_train  the training step of those blocks, with the gradients handed over as tac_stack_backward hands them
  backward  the backward call of one layer on recorded membranes

`net` names the network: `single` (one layer), `rate` (conv 1 -> c, mean pool, conv c -> 2c on rate-coded images),
`event` (Conv-LIF-MaxPool blocks of c channels on event frames, the pool applied by the layer that writes the spikes)
and `vgg` (2 -> c -> 2c -> 2c -> 4c -> 4c, stride 2 in the first, third and fifth layer).

Inputs are drawn on the GPU from the seed: rate-coded images (one rate per pixel, U[0,1]), event-camera frames (a
patch of rate 0.3 moving over a background of 0.02; real-valued frames carry normalised log counts) or independent
spikes at a fixed rate, with Kaiming-normal weights.
"""
import math

import torch

from paper_2603_13810_amd import api

DEVICE = "cuda:0"
MODES = {"per_step": api.TAC_PER_STEP, "TAC": api.TAC_COLLAPSE, "TAC_TP": api.TAC_PRESERVE}
# what a layer reads: packed bits, bits behind a 2 x 2 mean pool, real-valued frames
IN_FORMATS = {"bits": api.TAC_IN_BITS, "mean": api.TAC_IN_BITS_POOL2, "f32": api.TAC_IN_F32}


def _case(name, kind, net, **values):
    c = dict(kind=kind, net=net, spikes="bernoulli", rate=0.1, T=16, B=16, H=32, W=32, Cin=2, c=32, blocks=1, stride=1,
             mode="TAC", K=4, bf16=True, beta=0.9, bias=False, readout=False, detach=False, arctan=False,
             per_group=False)
    c.update(values)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one small fp32 layer on a handful of images: what a first experiment or an interactive call runs
        _case("small_layer", "layer", "single", spikes="rate", T=4, B=4, Cin=1, H=28, W=28, c=8, K=2, bf16=False),
        # the two-layer rate-coded network, inference at the training batch, spikes unpacked for the dense head
        _case("rate_net", "stack", "rate", spikes="rate", T=8, B=128, H=28, W=28, c=32, K=4, readout=True),
        # the same in fp32 on the 25 frames of the rate-coded runs, whose last group is shorter (25 = 3 x 8 + 1)
        _case("rate_net_fp32", "stack", "rate", spikes="rate", T=25, B=128, H=28, W=28, c=32, K=8, bf16=False),
        # event-camera frames as they leave a decoder (bytes), packed and run through the strided first layer
        _case("event_frames", "frames", "single", spikes="event", T=16, B=32, Cin=2, H=128, W=128, c=64, stride=2,
              mode="TAC_TP", K=2, beta=0.5),
        # the event-data network: five Conv-BN-LIF-MaxPool blocks, the first on normalised counts, the evaluation batch
        _case("event_net", "blocks", "event", spikes="counts", rate=0.15, T=16, B=16, H=64, W=64, c=128, blocks=5,
              mode="TAC_TP", K=4, beta=0.5, bias=True),
        # the five-layer strided stack on event frames
        _case("vgg_net", "stack", "vgg", spikes="event", T=16, B=16, H=128, W=128, c=64, mode="TAC_TP", K=2, beta=0.5),
        # a wide hidden layer at the largest batch: the roofline workload
        _case("wide_layer", "stack", "single", T=32, B=256, Cin=128, H=64, W=64, c=128, K=4),
        # the same layer with every frame's spikes kept, more active inputs, an ordinary batch
        _case("wide_layer_tp", "stack", "single", rate=0.2, T=32, B=64, Cin=128, H=64, W=64, c=128, mode="TAC_TP", K=8),
        # a hidden layer whose sizes are no powers of two, with a shorter last group (25 = 6 x 4 + 1) and a bias
        _case("odd_layer", "stack", "single", T=25, B=24, Cin=48, H=45, W=45, c=80, K=4, bias=True),
        # training step of the rate-coded network (fast sigmoid, slope 25, batch 128, 25 frames)
        _case("rate_train", "train", "rate", spikes="rate", T=25, B=128, H=28, W=28, c=32, K=4, bf16=False),
        # training step of the event-data network (arctan, slope 2, reset detached, batch 16)
        _case("event_train", "blocks_train", "event", spikes="counts", rate=0.15, T=16, B=16, H=64, W=64, c=128, blocks=5,
              mode="TAC_TP", K=4, beta=0.5, bias=True, detach=True, arctan=True),
        # backward call of the wide hidden layer inside a stack, its input gradient once per group
        _case("wide_backward", "backward", "single", T=32, B=64, Cin=128, H=64, W=64, c=128, K=4, per_group=True),
    ]


# ---- drawn cases -------------------------------------------------------------------------------

def _log_int(rng, low, high):
    return int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))


def _draw_one(rng):
    mode = rng.choice(["per_step", "TAC", "TAC", "TAC_TP", "TAC_TP"])
    K = 1 if mode == "per_step" else rng.choice([2, 2, 3, 4, 4, 5, 8, 8, 16])
    which = rng.randrange(11)
    if which == 0:                                              # small layers
        return _case(None, "layer", "single", spikes="rate", T=rng.randint(2, 25), B=_log_int(rng, 1, 16), Cin=rng.choice([1, 2]),
                     H=rng.randint(10, 34), W=rng.randint(10, 34), c=rng.choice([8, 12, 16, 32]), mode=mode, K=K, bf16=False)
    if which in (1, 2):                                         # rate-coded network, both precisions
        side = 2 * rng.randint(10, 17)
        return _case(None, "stack", "rate", spikes="rate", T=rng.randint(4, 25), B=_log_int(rng, 8, 256), H=side, W=side,
                     c=rng.choice([16, 24, 32, 40, 48]), mode=mode, K=K, bf16=which == 1, readout=rng.random() < 0.5)
    if which == 3:                                              # packed first layer on event frames
        return _case(None, "frames", "single", spikes="event", T=rng.randint(6, 32), B=_log_int(rng, 4, 48), Cin=2,
                     H=rng.randint(40, 128), W=rng.randint(40, 128), c=rng.choice([32, 48, 64, 128]), stride=rng.choice([1, 2]),
                     mode=mode, K=K, beta=0.5)
    if which == 4:                                              # event-data network
        side, blocks = rng.choice([(32, 4), (32, 5), (48, 4), (64, 5), (80, 4), (96, 5)])
        return _case(None, "blocks", "event", spikes=rng.choice(["counts", "event"]), rate=rng.uniform(0.05, 0.3),
                     T=rng.randint(6, 24), B=_log_int(rng, 2, 32), H=side, W=side, c=rng.choice([32, 48, 64, 96, 128]),
                     blocks=blocks, mode=mode, K=K, beta=0.5, bias=True)
    if which == 5:                                              # strided stack
        side = rng.choice([64, 80, 96, 100, 128])
        return _case(None, "stack", "vgg", spikes="event", T=rng.randint(6, 24), B=_log_int(rng, 2, 24), H=side, W=side,
                     c=rng.choice([16, 32, 48, 64]), mode=mode, K=K, beta=0.5)
    if which == 6:                                              # wide layers
        side = rng.choice([32, 32, 64, 64, 64, 28, 56])
        return _case(None, "stack", "single", rate=rng.uniform(0.05, 0.3), T=rng.randint(8, 32), B=_log_int(rng, 8, 128),
                     Cin=rng.choice([64, 96, 128]), H=side, W=side, c=rng.choice([128, 128, 256]), mode=mode, K=K)
    if which == 7:                                              # odd layers
        return _case(None, "stack", "single", rate=rng.uniform(0.05, 0.3), T=rng.randint(5, 25), B=_log_int(rng, 4, 48),
                     Cin=8 * rng.randint(1, 12), H=rng.randint(9, 60), W=rng.randint(9, 60), c=8 * rng.randint(2, 16), mode=mode,
                     K=K, bias=True)
    if which == 8:                                              # rate-coded training
        side = 2 * rng.randint(10, 16)
        return _case(None, "train", "rate", spikes="rate", T=rng.randint(4, 25), B=_log_int(rng, 16, 128), H=side, W=side,
                     c=rng.choice([16, 24, 32]), mode=mode, K=K, bf16=rng.random() < 0.3)
    if which == 9:                                              # event-data training
        side, blocks = rng.choice([(32, 4), (32, 5), (48, 4), (64, 5)])
        return _case(None, "blocks_train", "event", spikes=rng.choice(["counts", "event"]), rate=rng.uniform(0.05, 0.3),
                     T=rng.randint(6, 16), B=_log_int(rng, 2, 16), H=side, W=side, c=rng.choice([32, 64, 96, 128]),
                     blocks=blocks, mode=mode, K=K, beta=0.5, bias=True, detach=rng.random() < 0.5, arctan=True)
    return _case(None, "backward", "single", rate=rng.uniform(0.05, 0.3), T=rng.randint(6, 24), B=_log_int(rng, 4, 32),
                 Cin=rng.choice([32, 64, 96, 128]), H=rng.choice([32, 64, 32, 64, 24]), W=rng.choice([32, 64, 32, 64, 40]),
                 c=rng.choice([64, 128, 128]), mode=mode, K=K, arctan=rng.random() < 0.5, per_group=rng.random() < 0.5)


def draw(rng):
    """Another case of the listed ranges.  The largest products are taken at a smaller batch: a drawn training or
    backward case holds at most 0.2 TFLOP, any other at most 1."""
    c = _draw_one(rng)
    while c["B"] > 1 and work(c)["flops"] > (2e11 if c["kind"] in ("train", "blocks_train", "backward") else 1e12):
        c["B"] = max(1, c["B"] // 2)
    return c


# ---- the network of a case ---------------------------------------------------------------------

def _descs(c):
    """The layers as descriptions of the C ABI."""
    T, H, W = c["T"], c["H"], c["W"]
    first = "f32" if c["spikes"] == "counts" else "bits"
    width = c["c"]
    if c["net"] == "single":
        spec = [(c["Cin"], width, c["stride"], first, False)]
    elif c["net"] == "rate":
        spec = [(1, width, 1, first, False), (width, 2 * width, 1, "mean", False)]
    elif c["net"] == "event":
        spec = [(2 if i == 0 else width, width, 1, first if i == 0 else "bits", True) for i in range(c["blocks"])]
    else:
        chans = [2, width, 2 * width, 2 * width, 4 * width, 4 * width]
        spec = [(chans[i], chans[i + 1], 2 - i % 2, first if i == 0 else "bits", False) for i in range(5)]
    descs = []
    for Cin, Cout, stride, load, pooled in spec:
        if load == "mean":
            H, W = H // 2, W // 2
        d = api.make_desc(T, c["B"], Cin, H, W, Cout, K=c["K"], beta=c["beta"], theta=1.0, mode=MODES[c["mode"]], stride=stride,
                          precision=api.TAC_BF16 if c["bf16"] else api.TAC_FP32, in_format=IN_FORMATS[load],
                          out_format=api.TAC_OUT_BITS_MAXPOOL2 if pooled else api.TAC_OUT_BITS)
        descs.append(d)
        T, Ho, Wo = _out_shape(d)
        H, W = (Ho // 2, Wo // 2) if pooled else (Ho, Wo)
    return descs


def _group(d):
    """(frames per group, number of groups)."""
    K = 1 if d.mode == api.TAC_PER_STEP else min(d.K, d.T)
    return K, -(-d.T // K)


def _out_shape(d):
    Ho, Wo = (d.H - 1) // d.stride + 1, (d.W - 1) // d.stride + 1
    return (_group(d)[1] if d.mode == api.TAC_COLLAPSE else d.T), Ho, Wo


def _stored_shape(d):
    T_out, Ho, Wo = _out_shape(d)
    return (T_out, Ho // 2, Wo // 2) if d.out_format == api.TAC_OUT_BITS_MAXPOOL2 else (T_out, Ho, Wo)


# ---- inputs ------------------------------------------------------------------------------------

def _rng(seed, stream):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(int(seed) * 1000 + stream)
    return g


def _frames(c, d, i, seed):
    """The T input frames [B, Cin, H, W] of layer i one after the other: 0/1 bytes, or float32 counts.  Hidden layers that
    are run on spikes of their own get independent ones at the case's rate."""
    g = _rng(seed, 10 + i)
    f = 2 if d.in_format == api.TAC_IN_BITS_POOL2 else 1
    T, B, Cin, H, W = d.T, d.B, d.Cin, f * d.H, f * d.W
    spikes = c["spikes"] if i == 0 else "bernoulli"
    p = torch.rand((B, Cin, H, W), generator=g, device=DEVICE) if spikes == "rate" else c["rate"]
    phi = torch.rand((B, 1, 1), generator=g, device=DEVICE) * (2 * math.pi)
    ys = torch.arange(H, device=DEVICE).view(1, H, 1)
    xs = torch.arange(W, device=DEVICE).view(1, 1, W)
    patch = 24 * min(H, W) // 128 + 1
    for t in range(T):
        u = torch.rand((B, Cin, H, W), generator=g, device=DEVICE)
        if spikes in ("rate", "bernoulli"):
            yield (u < p).to(torch.uint8)
            continue
        s = (t - (T - 1) / 2) * 4.0 * min(H, W) / 128
        cy, cx = torch.round(H / 2 + s * torch.sin(phi)), torch.round(W / 2 + s * torch.cos(phi))
        inside = ((ys - cy).abs() <= patch // 2) & ((xs - cx).abs() <= patch // 2)
        hit = u < torch.where(inside, 0.3, 0.02).view(B, 1, H, W)
        if spikes == "event":
            yield hit.to(torch.uint8)
        else:                                                   # log(1 + f) / log(1 + f_max), f_max = 8 events per pixel
            f = torch.randint(1, 9, (B, Cin, H, W), generator=g, device=DEVICE).float()
            yield torch.where(hit, torch.log1p(f) / math.log(9.0), 0.0)


def _input(c, d, i, seed):
    """What layer i reads: packed words, or real-valued frames."""
    frames = _frames(c, d, i, seed)
    if d.in_format == api.TAC_IN_F32:
        return torch.stack(list(frames))
    return torch.stack([api.tac_pack_spikes(f) for f in frames])


def _weights(c, seed):
    g = _rng(seed, 1)
    out = []
    for d in _descs(c):
        w = torch.randn((d.Cout, d.Cin, 3, 3), generator=g, device=DEVICE) * math.sqrt(2.0 / (9 * d.Cin))
        b = torch.randn((d.Cout,), generator=g, device=DEVICE) * 0.1 if c["bias"] else None
        out.append((w, b))
    return out


def _gradient(shape, seed, i=0):
    return torch.randn(shape, generator=_rng(seed, 30 + i), device=DEVICE)


def _next_group(descs, i):
    """Output steps of layer i that share one gradient: the group of the layer behind it (0: none)."""
    K = _group(descs[i + 1])[0] if i + 1 < len(descs) else 1
    return K if K > 1 else 0


def _backward_options(c):
    return dict(surrogate=api.TAC_SG_ARCTAN if c["arctan"] else api.TAC_SG_FAST_SIGMOID, alpha=2.0 if c["arctan"] else 25.0,
                detach_reset=c["detach"])


def _membranes(d, seed):
    """Membranes before the reset as a layer records them: the recurrence under normally distributed input currents,
    of the spread that the convolution of Kaiming weights with these spikes has."""
    g = _rng(seed, 3)
    K, G = _group(d)
    T_out, Ho, Wo = _out_shape(d)
    trace = torch.empty((T_out, d.B, d.Cout, Ho, Wo), device=DEVICE)
    v = torch.zeros((d.B, d.Cout, Ho, Wo), device=DEVICE)
    n = 0
    for k in range(G):
        Kg = min(K, d.T - k * K)
        y = torch.randn((d.B, d.Cout, Ho, Wo), generator=g, device=DEVICE) * (0.45 * math.sqrt(Kg))
        for _ in range(Kg if d.mode == api.TAC_PRESERVE else 1):
            v = v * (d.beta ** Kg if d.mode == api.TAC_COLLAPSE else d.beta) + y
            trace[n] = v
            v = v - (v >= d.theta).float() * d.theta
            n += 1
    return trace


def prepare(case, seed):
    c = case
    kind, descs = c["kind"], _descs(c)
    weights = _weights(c, seed)
    s = dict(kind=kind, descs=descs, weights=weights, options=_backward_options(c))
    if kind == "backward":
        d = descs[0]
        T_out, Ho, Wo = _out_shape(d)
        s["input"] = _input(c, d, 0, seed)
        s["trace"] = _membranes(d, seed)
        s["grad_out"] = _gradient((T_out, d.B, d.Cout, Ho, Wo), seed)
        s["options"]["grad_in_per_group"] = c["per_group"]
        return s
    if kind == "frames":
        d = descs[0]
        s["dense"] = torch.stack(list(_frames(c, d, 0, seed)))
        s["packed"] = torch.empty((d.T, d.B, d.Cin, d.H, (d.W + 31) // 32), dtype=torch.int32, device=DEVICE)
    elif kind in ("blocks", "blocks_train"):
        s["inputs"] = [_input(c, d, i, seed) for i, d in enumerate(descs)]
    else:
        s["input"] = _input(c, descs[0], 0, seed)
    # a layer with a shorter last group carries its membrane through a buffer of the caller, as streaming calls do; one
    # allocation holds them all, so that a new sequence starts with one fill
    ragged = [d.T % _group(d)[0] != 0 or kind == "layer" for d in descs]
    sizes = [d.B * d.Cout * _out_shape(d)[1] * _out_shape(d)[2] if r else 0 for d, r in zip(descs, ragged)]
    s["state"] = torch.zeros((sum(sizes),), device=DEVICE) if sum(sizes) else None
    s["layers"], at = [], 0
    for d, (w, b), n in zip(descs, weights, sizes):
        T_out, Ho, Wo = _out_shape(d)
        Ts, Hs, Ws = _stored_shape(d)
        L = dict(desc=d, w_prepared=api.tac_prepare_weights(d, w), bias=b,
                 out_spikes_packed=torch.empty((Ts, d.B, d.Cout, Hs, (Ws + 31) // 32), dtype=torch.int32, device=DEVICE))
        if n:
            L["v_inout"] = s["state"][at:at + n].view(d.B, d.Cout, Ho, Wo)
            at += n
        if kind in ("train", "blocks_train"):
            L["v_trace"] = torch.empty((T_out, d.B, d.Cout, Ho, Wo), device=DEVICE)
        s["layers"].append(L)
    if kind in ("stack", "train"):
        s["stack"], s["outs"] = api.make_stack(s["layers"])
        s["readout"] = _stored_shape(descs[-1])[2] if c["readout"] else 0
    if kind == "train":
        Ts, Hs, Ws = _stored_shape(descs[-1])
        s["grad_out"] = _gradient((Ts, c["B"], descs[-1].Cout, Hs, Ws), seed)
    if kind == "blocks_train":
        s["grad_out"] = []
        for i, d in enumerate(descs):
            Ts, Hs, Ws = _stored_shape(d)
            Kc = _next_group(descs, i)
            s["grad_out"].append(_gradient((-(-Ts // Kc) if Kc else Ts, d.B, d.Cout, Hs, Ws), seed, i))
    return s


def _layer_call(L, x):
    return api.tac_conv_lif(L["desc"], x, L["w_prepared"], L["bias"], L.get("v_inout"), L["out_spikes_packed"], L.get("v_trace"))


def run(state):
    s = state
    kind = s["kind"]
    if kind == "backward":
        return api.tac_conv_lif_backward(s["descs"][0], s["input"], s["weights"][0][0], s["trace"], s["grad_out"], **s["options"])
    if s["state"] is not None:
        s["state"].zero_()                                      # a new sequence starts from rest
    if kind == "layer":
        return dict(spikes=_layer_call(s["layers"][0], s["input"]), v=s["layers"][0]["v_inout"])
    if kind == "frames":
        x = api.tac_pack_spikes(s["dense"], s["packed"])
        return dict(spikes=_layer_call(s["layers"][0], x), packed=x)
    if kind in ("train", "blocks_train"):
        for L, (w, _) in zip(s["layers"], s["weights"]):
            api.tac_prepare_weights(L["desc"], w, L["w_prepared"])
    if kind in ("blocks", "blocks_train"):
        spikes = [_layer_call(L, x) for L, x in zip(s["layers"], s["inputs"])]
        if kind == "blocks":
            return dict(spikes=spikes)
        grads = []
        for i in reversed(range(len(spikes))):
            g = api.tac_conv_lif_backward(s["descs"][i], s["inputs"][i], s["weights"][i][0], s["layers"][i]["v_trace"], s["grad_out"][i],
                                          want_input_grad=i > 0, grad_in_per_group=True, grad_out_group_K=_next_group(s["descs"], i),
                                          grad_out_group_beta=s["descs"][i].beta, **s["options"])
            grads.insert(0, dict(w=g["grad_w"], bias=g["grad_bias"], input=g["grad_in"]))
        return dict(spikes=spikes, grads=grads)
    api.tac_stack_forward(s["stack"], s["input"])
    if kind == "train":
        grads = api.tac_stack_backward(s["stack"], [w for w, _ in s["weights"]], s["input"], s["grad_out"], grad_in_per_group=True,
                                       **s["options"])
        return dict(spikes=s["outs"][-1], grads=[dict(w=g["grad_w"], bias=g["grad_bias"]) for g in grads])
    if s["readout"]:
        return dict(spikes=s["outs"], dense=api.tac_unpack_spikes(s["outs"][-1], s["readout"]))
    return dict(spikes=s["outs"])


# ---- what a pass cannot do without -------------------------------------------------------------

def work(case):
    """Every input read once, every output written once; the multiplications of the convolutions (T / K stages) and, where
    gradients are asked for, of their weight gradients and of the input gradients that a layer before needs."""
    c = case
    kind, descs = c["kind"], _descs(c)
    by_block = kind in ("blocks", "blocks_train")
    training = kind in ("train", "blocks_train")
    bytes_ = flops = 0
    for i, d in enumerate(descs):
        T_out, Ho, Wo = _out_shape(d)
        Ts, Hs, Ws = _stored_shape(d)
        G = _group(d)[1]
        conv = 2 * G * d.B * Ho * Wo * d.Cout * d.Cin * 9
        n_w = d.Cout * d.Cin * 9
        out = 4 * Ts * d.B * d.Cout * Hs * ((Ws + 31) // 32)
        if i == 0 or by_block:
            bytes_ += d.T * d.B * d.Cin * d.H * (4 * d.W if d.in_format == api.TAC_IN_F32 else 4 * ((d.W + 31) // 32))
        if kind == "backward":
            flops += 2 * conv
            bytes_ += 4 * (2 * T_out * d.B * d.Cout * Ho * Wo + G * d.B * d.Cout * Ho * Wo +
                           (G if c["per_group"] else d.T) * d.B * d.Cin * d.H * d.W + 2 * n_w)
            continue
        flops += conv * (1 if not training else 2 if i == 0 else 3)
        bytes_ += out + n_w * (8 if training else 2 if c["bf16"] else 4)
        if training and (by_block or i == len(descs) - 1):       # the gradient of the spikes that the layer stored
            Kc = _next_group(descs, i) or 1
            bytes_ += 4 * -(-Ts // Kc) * d.B * d.Cout * Hs * Ws
        if kind == "blocks_train" and i > 0:
            bytes_ += 4 * G * d.B * d.Cin * d.H * d.W
        if kind == "layer":
            bytes_ += 8 * d.B * d.Cout * Ho * Wo
        if kind == "frames":
            bytes_ += d.T * d.B * d.Cin * d.H * d.W
    if c["readout"]:
        bytes_ += Ts * d.B * d.Cout * Hs * Ws
    return dict(bytes=bytes_, flops=flops)


def tolerance(case):
    """Sums in another order move a membrane in its last bits; where that crosses the threshold a spike flips and the
    neuron's later steps follow, so spikes are compared by the share of packed words that differ: at most 7.5e-6 between
    the vector kernel and the matrix-core kernels on these networks, but one word in the smallest outputs is 1e-3 of them.
    Gradients: 1.7e-5 between the two in a fp32 training step (a surrogate of slope 25 on membranes that differ in their
    last bits), 2.4e-3 where a bf16 layer's gradients multiply rounded operands, 5e-7 on the same membranes in fp32."""
    if case["kind"] == "backward":
        return dict(rel=1e-2 if case["bf16"] else 1e-5)
    if case["kind"] in ("train", "blocks_train"):
        return dict(rel=1e-2 if case["bf16"] else 2e-4, differ=1e-3)
    if case["kind"] == "layer":
        return dict(rel=1e-5, max=1e-3, differ=1e-4)
    return dict(rel=0.0, differ=1e-3)


# ---- the same in 64 bits -----------------------------------------------------------------------

def _shifted(a, ky, kx, stride, Ho, Wo):
    """The input pixels under tap (ky, kx) of every output, from a zero-padded tensor: [B, Cin, Ho Wo]."""
    v = a[:, :, ky:ky + (Ho - 1) * stride + 1:stride, kx:kx + (Wo - 1) * stride + 1:stride]
    return v.reshape(v.shape[0], v.shape[1], Ho * Wo)


def _conv64(a, w, stride):
    B, _, H, W = a.shape
    Ho, Wo = (H - 1) // stride + 1, (W - 1) // stride + 1
    pad = torch.nn.functional.pad(a, (1, 1, 1, 1))
    y = torch.zeros((B, w.shape[0], Ho * Wo), dtype=torch.float64, device=a.device)
    for ky in range(3):
        for kx in range(3):
            y += torch.matmul(w[:, :, ky, kx].contiguous(), _shifted(pad, ky, kx, stride, Ho, Wo))
    return y.view(B, -1, Ho, Wo)


def _conv64_gradients(a, w, gy, stride, want_input):
    """Weight and input gradient of _conv64."""
    B, Cin, H, W = a.shape
    Ho, Wo = gy.shape[2], gy.shape[3]
    pad = torch.nn.functional.pad(a, (1, 1, 1, 1))
    flat = gy.reshape(B, gy.shape[1], Ho * Wo)
    gw = torch.zeros_like(w)
    gp = torch.zeros_like(pad) if want_input else None
    for ky in range(3):
        for kx in range(3):
            x = _shifted(pad, ky, kx, stride, Ho, Wo)
            gw[:, :, ky, kx] = torch.matmul(flat, x.transpose(1, 2).contiguous()).sum(0)
            if want_input:
                part = torch.matmul(w[:, :, ky, kx].t().contiguous(), flat).view(B, Cin, Ho, Wo)
                gp[:, :, ky:ky + (Ho - 1) * stride + 1:stride, kx:kx + (Wo - 1) * stride + 1:stride] += part
    return gw, gp[:, :, 1:-1, 1:-1] if want_input else None


def _aggregates64(d, frames):
    """A_k of every group of frames (an iterator), in 64 bits, the mean pool on load applied."""
    K, G = _group(d)
    frames = iter(frames)
    for k in range(G):
        Kg = min(K, d.T - k * K)
        a = 0.0
        for j in range(Kg):
            x = next(frames).double()
            if d.in_format == api.TAC_IN_BITS_POOL2:
                x = torch.nn.functional.avg_pool2d(x, 2)
            a = a + d.beta ** (Kg - 1 - j) * x
        yield Kg, a


def _forward64(d, frames, w, b, trace=None):
    """Spikes of every output step (bytes, before a pool in the writer) and the last membrane; `trace` collects membranes.
    With bf16 operands weights and aggregates are rounded, as the entry point says, and everything else is in 64 bits."""
    v, out = 0.0, []
    rounded = (lambda x: x.to(torch.bfloat16).double()) if d.precision == api.TAC_BF16 else (lambda x: x.double())
    w64 = rounded(w)
    for Kg, a in _aggregates64(d, frames):
        a = rounded(a)
        y = torch.cat([_conv64(part, w64, d.stride) for part in a.split(max(1, (1 << 26) // (d.Cin * d.H * d.W)))])
        if b is not None:
            y = y + b.double().view(1, -1, 1, 1)
        for _ in range(Kg if d.mode == api.TAC_PRESERVE else 1):
            v = (d.beta ** Kg if d.mode == api.TAC_COLLAPSE else d.beta) * v + y
            if trace is not None:
                trace.append(v)
            s = v >= d.theta
            out.append(s.to(torch.uint8))
            v = v - s.double() * d.theta
    return out, v


def _pooled(d, spikes):
    if d.out_format != api.TAC_OUT_BITS_MAXPOOL2:
        return spikes
    return [torch.nn.functional.max_pool2d(s.float(), 2).to(torch.uint8) for s in spikes]


def _packed(spikes):
    """int32 words [T, ..., ceil(W / 32)] of 0/1 bytes."""
    words = []
    for s in spikes:
        s = torch.nn.functional.pad(s, (0, -s.shape[-1] % 32))
        bits = s.view(*s.shape[:-1], -1, 32).to(torch.int64) << torch.arange(32, device=s.device)
        total = bits.sum(-1)
        words.append(torch.where(total >= 2 ** 31, total - 2 ** 32, total).to(torch.int32))
    return torch.stack(words)


def _surrogate64(c, x):
    if c["arctan"]:
        return 1.0 / (1.0 + (math.pi * x) ** 2)                 # (alpha / 2) / (1 + (pi alpha x / 2)^2), alpha = 2
    return 1.0 / (1.0 + 25.0 * x.abs()) ** 2


def _backward64(c, d, frames, w, trace, grad_out, want_input, per_group):
    """Gradients of one layer; trace and grad_out are sequences over its output steps (grad_out before a pool in the writer)."""
    K, G = _group(d)
    carry, gys, n = 0.0, [None] * G, len(trace)
    for k in reversed(range(G)):
        Kg = min(K, d.T - k * K)
        total = 0.0
        for _ in range(Kg if d.mode == api.TAC_PRESERVE else 1):
            n -= 1
            sg = _surrogate64(c, trace[n].double() - d.theta)
            gv = grad_out[n].double() * sg + carry * (1.0 if c["detach"] else 1.0 - d.theta * sg)
            total = total + gv
            carry = (d.beta ** Kg if d.mode == api.TAC_COLLAPSE else d.beta) * gv
        gys[k] = total
    w64 = w.double()
    gw, gin = torch.zeros_like(w64), []
    for (Kg, a), gy in zip(_aggregates64(d, frames), gys):
        step = max(1, (1 << 26) // (max(d.Cin, d.Cout) * d.H * d.W))
        parts = [_conv64_gradients(x, w64, y, d.stride, want_input) for x, y in zip(a.split(step), gy.split(step))]
        gw += sum(p[0] for p in parts)
        if want_input:
            g = torch.cat([p[1] for p in parts])
            gin += [g] if per_group else [d.beta ** (Kg - 1 - j) * g for j in range(Kg)]
    return dict(grad_y=torch.stack(gys), grad_w=gw, grad_bias=sum(g.sum((0, 2, 3)) for g in gys), grad_in=gin)


def _through_pool(d, spikes, grad):
    """Gradient of the pooled spikes to the first maximal spike of each window, in row-major order."""
    if d.out_format != api.TAC_OUT_BITS_MAXPOOL2:
        return grad
    B, C, H, W = spikes.shape
    win = spikes.view(B, C, H // 2, 2, W // 2, 2).permute(0, 1, 2, 4, 3, 5).reshape(B, C, H // 2, W // 2, 4)
    order = win * torch.tensor([8, 6, 4, 2], device=win.device) + torch.tensor([1, 0, 0, 0], device=win.device)
    first = order.argmax(-1, keepdim=True)                      # the first pixel where none has spiked
    g = torch.zeros(win.shape, dtype=torch.float64, device=win.device).scatter_(-1, first, grad.double().unsqueeze(-1))
    return g.view(B, C, H // 2, W // 2, 2, 2).permute(0, 1, 2, 4, 3, 5).reshape(B, C, H, W)


def exact(case, seed):
    c = case
    kind, descs = c["kind"], _descs(c)
    weights = _weights(c, seed)
    d = descs[0]
    if kind == "backward":
        T_out, Ho, Wo = _out_shape(d)
        grad_out = _gradient((T_out, d.B, d.Cout, Ho, Wo), seed)
        r = _backward64(c, d, _frames(c, d, 0, seed), weights[0][0], _membranes(d, seed), grad_out, True, c["per_group"])
        r["grad_in"] = torch.stack(r["grad_in"])
        return r
    by_block = kind in ("blocks", "blocks_train")
    training = kind in ("train", "blocks_train")
    outs, traces, inputs = [], [], []
    for i, (d, (w, b)) in enumerate(zip(descs, weights)):
        if i == 0 or by_block:
            frames = _frames(c, d, i, seed)
            frames = list(frames) if kind != "stack" else frames
        trace = [] if training else None
        spikes, v = _forward64(d, frames, w, b, trace)
        inputs.append(frames)
        traces.append((trace, spikes))
        frames = _pooled(d, spikes)
        outs.append(_packed(frames))
    if kind == "layer":
        return dict(spikes=outs[0], v=v)
    if kind == "frames":
        return dict(spikes=outs[0], packed=_packed(inputs[0]))
    if not training:
        return dict(spikes=outs, dense=torch.stack(frames)) if c["readout"] else dict(spikes=outs)
    grads = []
    for i in reversed(range(len(descs))):
        d, (trace, spikes) = descs[i], traces[i]
        Ts, Hs, Ws = _stored_shape(d)
        if by_block:
            Kc = _next_group(descs, i)
            g = _gradient((-(-Ts // Kc) if Kc else Ts, d.B, d.Cout, Hs, Ws), seed, i).double()
            # the K steps of a group of the next layer share its gradient, weighted by that layer's decay
            grad = [g[n // Kc] * d.beta ** (min(Kc, Ts - n // Kc * Kc) - 1 - n % Kc) for n in range(Ts)] if Kc else list(g)
        elif i == len(descs) - 1:
            grad = list(_gradient((Ts, d.B, d.Cout, Hs, Ws), seed))
        grad = [_through_pool(d, x, g) for x, g in zip(spikes, grad)]
        r = _backward64(c, d, inputs[i], weights[i][0], trace, grad, i > 0, by_block)
        grads.insert(0, dict(w=r["grad_w"], bias=r["grad_bias"]))
        if by_block:
            grads[0]["input"] = torch.stack(r["grad_in"]) if i > 0 else None
        grad = r["grad_in"]
        if d.in_format == api.TAC_IN_BITS_POOL2:                # a quarter to each input of the mean pool
            grad = [0.25 * g.repeat_interleave(2, 2).repeat_interleave(2, 3) for g in grad]
    return dict(spikes=outs if by_block else outs[-1], grads=grads)
