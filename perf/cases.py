"""What this library is timed on: the work its users have it do, through its public entry points.

Two kinds of case.

* "block": 3x3x3 convolution layers (ReLU between them) on a tile grid through the C-ABI binding, as a program does
  that brings its own network around the layers: partition the volume, give every layer input its margins, convolve,
  reassemble; with steps = "all" also the backward pass (data gradients, weight and bias gradients).  `exchange` says
  how the margins arrive: "messages" (halo_pack + halo_unpack, what devices that send each other messages do), "pass"
  (sp_halo_exchange) or "gather" (the convolutions read the neighbour tiles themselves where they can).
* "net": the U-Net driver.  steps = "all" is a training step (forward, Dice + cross-entropy loss, backward: logits, loss
  and every weight gradient come back), "forward" is inference (logits).  flat = True is the 2-D network on slabs.

Sizes are those of the workload list, the benchmark and the tests, plus ragged ones in between.  Inputs: CT-like
single-channel volumes for the networks and first layers, N(0, 1) activations and upstream gradients, random weights.
"""
import math

import torch

from paper_1909_03108_amd import sp3d, unet

KEEP = sp3d.SP_HALO_SKIP_SEND | sp3d.SP_HALO_KEEP_ZERO


def _block(name, dtype, dhw, grid, channels, steps, exchange, relu_last=False, n=1):
    return dict(name=name, kind="block", dtype=dtype, n=n, d=dhw[0], h=dhw[1], w=dhw[2], gd=grid[0], gh=grid[1],
                gw=grid[2], channels=channels, steps=steps, exchange=exchange, relu_last=relu_last)


def _net(name, dhw, grid, channels, convs, steps, in_ch=1, flat=False, gather=False, bits=False, coarse="", n=1):
    return dict(name=name, kind="net", dtype="bf16", n=n, d=dhw[0], h=dhw[1], w=dhw[2], gd=grid[0], gh=grid[1],
                gw=grid[2], channels=channels, convs=convs, steps=steps, in_ch=in_ch, classes=3, flat=flat,
                gather=gather, bits=bits, coarse=coarse)


FOUR, SIX = "32,64,128,256", "32,64,128,256,512,1024"


def listed():
    return [
        # the smallest call of the workload list: one fp32 layer on 32^3, forward only (launches and latency)
        _block("layer_f32_32", "f32", (32, 32, 32), (2, 2, 1), "8,16", "forward", "pass"),
        # fp32 training of a narrow pair of layers on an odd-sized patch (numerics checks, small research networks)
        _block("pair_f32_odd", "f32", (51, 62, 70), (1, 2, 2), "8,16,16", "all", "pass", True),
        # the workload list's pair of 32-channel layers on 128^3: forward and backward
        _block("pair_128", "bf16", (128, 128, 128), (4, 4, 1), "32,32,32", "all", "pass"),
        # first level of a U-Net on a 256^3 CT volume: 1 -> 32 -> 32 channels
        _block("level_256", "bf16", (256, 256, 256), (4, 4, 2), "1,32,32", "all", "gather", True),
        # first level on a three-phase scan of ragged extents: 3 -> 32 -> 32 channels
        _block("level_phases_ragged", "bf16", (99, 156, 210), (1, 2, 2), "3,32,32", "all", "pass", True),
        # the headline benchmark: one 32 -> 32 layer at 512^3, messages packed and unpacked, forward and backward
        _block("layer_512", "bf16", (512, 512, 512), (4, 4, 1), "32,32", "all", "messages"),
        # a training step on a small patch (the tests' size): launches and host work count
        _net("net3d_train_32", (32, 32, 32), (2, 2, 1), FOUR, 2, "all"),
        # inference on a ragged clinical volume
        _net("net3d_infer_ragged", (112, 176, 208), (2, 2, 1), FOUR, 2, "forward", gather=True),
        # the workload list's four-level U-Net at 256^3: a training step
        _net("net3d_train_256", (256, 256, 256), (4, 4, 1), FOUR, 2, "all"),
        # the paper's six-level network with four convolutions per block, at 256^3, with the driver's options on
        _net("net3d_paper_256", (256, 256, 256), (4, 4, 1), SIX, 4, "all", gather=True, bits=True, coarse="2,2,1"),
        # the paper's 2-D network on a batch of 16 slabs of 512 x 512 x 5: a training step
        _net("net2d_train_16", (16, 512, 512), (1, 2, 2), SIX, 4, "all", in_ch=5, flat=True),
        # ... and inference on two slabs at a time
        _net("net2d_infer_2", (2, 512, 512), (1, 2, 2), SIX, 4, "forward", in_ch=5, flat=True),
    ]


MOST_BLOCK_FLOPS, MOST_NET_FLOPS, MOST_NET2D_FLOPS = 22e12, 40e12, 10.5e12


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _draw(rng):
    pick = rng.random()
    if pick < 0.5:
        f32 = rng.random() < 0.35
        grid = (rng.choice([1, 2, 4]), rng.choice([1, 2, 4]), rng.choice([1, 1, 2]))
        edge = _log(rng, 24, 100) if f32 else _log(rng, 40, 480)
        dhw = tuple(max(2, round(edge * _log(rng, 0.7, 1.4) / g)) * g for g in grid)
        channels = rng.choice(["8,16", "8,16,16", "4,8", "16,16", "1,8,16", "32,32"] if f32 else
                              ["32,32", "32,32,32", "1,32,32", "3,32,32", "4,32", "32,64", "64,64", "64,64,64"])
        steps = rng.choice(["all", "all", "forward"])
        case = _block("", "f32" if f32 else "bf16", dhw, grid, channels, steps,
                      rng.choice(["messages", "pass", "pass"] if f32 else ["messages", "pass", "gather"]),
                      rng.random() < 0.5, rng.choice([1, 1, 2]) if edge < 100 else 1)
    elif pick < 0.8:
        six = rng.random() < 0.3
        channels, convs = (SIX, 4) if six else (rng.choice([FOUR, FOUR, "32,64,128"]), 2)
        least = 2 ** (channels.count(","))
        grid = rng.choice([(1, 1, 1), (2, 2, 1), (2, 2, 2)] if six else [(1, 1, 1), (2, 2, 1), (2, 2, 2), (4, 4, 1)])
        edge = _log(rng, 2 * least, 256)
        dhw = tuple(max(1, round(edge * _log(rng, 0.7, 1.4) / g / least)) * g * least for g in grid)
        gather = rng.random() < 0.5
        case = _net("", dhw, grid, channels, convs, rng.choice(["all", "all", "forward"]), gather=gather,
                    bits=gather and rng.random() < 0.5)
    else:
        channels, convs = rng.choice([(SIX, 4), (FOUR, 2)])
        least = 2 ** (channels.count(","))
        grid = rng.choice([(1, 1, 1), (1, 1, 2), (1, 2, 2), (1, 4, 4)])
        edge = _log(rng, 128, 512)
        dhw = (round(_log(rng, 1, 16)),) + tuple(max(1, round(edge / g / least)) * g * least for g in grid[1:])
        case = _net("", dhw, grid, channels, convs, rng.choice(["all", "all", "forward"]), in_ch=rng.choice([1, 3, 5]),
                    flat=True)
    del case["name"]
    return case


def draw(rng):
    """One more case of the same ranges, within the largest listed one's cost."""
    while True:
        case = _draw(rng)
        most = MOST_BLOCK_FLOPS if case["kind"] == "block" else (MOST_NET2D_FLOPS if case["flat"] else MOST_NET_FLOPS)
        if case["dtype"] == "f32":
            most = 5e10
        if work(case)["flops"] <= most and all(case[k] // case[g] >= 1 for k, g in (("d", "gd"), ("h", "gh"), ("w", "gw"))):
            return case


# ---- what one pass cannot do without ------------------------------------------------------------------------------

def _channels(case):
    return tuple(int(c) for c in case["channels"].split(","))


def _image(ch):
    """a few input channels are an image: nobody asks for the gradient with respect to it"""
    return ch[0] <= 4


def _layers(case):
    """(flops of the forward pass, whether its data gradient is needed, output elements) of every layer, in order."""
    vox = case["n"] * case["d"] * case["h"] * case["w"]
    if case["kind"] == "block":
        ch = _channels(case)
        return [(54.0 * ci * co * vox, i > 0 or not _image(ch), vox * co) for i, (ci, co) in enumerate(zip(ch, ch[1:]))]
    out, nd = [], 2 if case["flat"] else 3
    for name, shape in unet.layer_plan(_channels(case), case["in_ch"], case["classes"], case["convs"], flat=case["flat"]):
        v = vox if name == "head" else vox >> (nd * int(name[-1] if name[:2] == "up" else name[3]))
        taps = math.prod(shape[:nd]) if name[:2] != "up" else 1        # an up-sampled voxel sees one of the 2^nd taps
        out.append((2.0 * taps * shape[-2] * shape[-1] * v, name != "enc0_a", v * shape[-1]))
    return out


def work(case):
    """Bytes: input, upstream gradient or labels, weights and results once, and in a pass with a backward half every
    inner activation once out and once in.  Flops: the products of every convolution."""
    es = 4 if case["dtype"] == "f32" else 2
    vox = case["n"] * case["d"] * case["h"] * case["w"]
    layers, train = _layers(case), case["steps"] == "all"
    flops = sum(f * ((3 if dg else 2) if train else 1) for f, dg, _ in layers)
    if case["kind"] == "block":
        ch = _channels(case)
        weights = sum(27 * ci * co for ci, co in zip(ch, ch[1:]))
        nbytes = es * (vox * (ch[0] + ch[-1]) + weights)
        if train:
            nbytes += es * vox * (ch[-1] + (0 if _image(ch) else ch[0])) + 4 * weights
    else:
        plan = unet.layer_plan(_channels(case), case["in_ch"], case["classes"], case["convs"], flat=case["flat"])
        weights = sum(math.prod(shape) for _, shape in plan)
        nbytes = es * (vox * (case["in_ch"] + case["classes"]) + weights)
        if train:
            nbytes += es * vox + 4 * weights
    if train:
        nbytes += 2 * es * sum(e for _, _, e in layers[:-1])
    return {"bytes": float(nbytes), "flops": flops}


def tolerance(case):
    """About four times the largest error against the same pass with its sums in another order (hidden channels
    permuted), measured over the listed cases and 24 drawn ones.

    fp32: 3e-7 (norm) and 3e-6 (single values); behind a ReLU, a sum within a rounding of zero may be kept by one
    implementation and dropped by the other: at 3e-7 one in ten million, and a gradient with one such element among
    1e6 is off by 1e-3 in norm and by its full size there.
    bf16 layers: 2e-3, a rounding to bf16 per stored tensor and ReLUs decided the other way (0.43 in a single value).
    Networks: 6e-3 and 0.17, such roundings carried through every later layer."""
    relu = case["kind"] == "net" or case["relu_last"] or case["channels"].count(",") > 1
    if case["dtype"] == "f32":
        return {"rel": 1e-3, "max": 0.99} if relu and case["steps"] == "all" else {"rel": 2e-6, "max": 2e-5}
    if case["kind"] == "block":
        return {"rel": 8e-3, "max": 0.99} if relu and case["steps"] == "all" else {"rel": 1e-3, "max": 0.05}
    return {"rel": 2e-2, "max": 0.7}


# ---- inputs ---------------------------------------------------------------------------------------------------------

def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _normal(gen, shape, dtype, std=1.0, mean=0.0):
    """N(mean, std^2), drawn in pieces so that a 512^3 tensor needs no second copy of itself in fp32"""
    out = torch.empty(shape, dtype=dtype, device="cuda")
    flat = out.view(-1)
    step = 1 << 28
    for i in range(0, flat.numel(), step):
        part = flat[i:i + step]
        part.copy_(torch.randn(part.shape, generator=gen, device="cuda").mul_(std).add_(mean))
    return out


def _ct(gen, n, dhw, c):
    """CT-like volume in [-1, 1] (uniform Hounsfield-like noise and eight Gaussian blobs), fp32, and its blobs alone"""
    D, H, W = dhw
    noise = torch.rand((n, D, H, W, c), generator=gen, device="cuda") * 2.0 - 1.0
    par = torch.rand((8, 6), generator=gen, device="cuda")
    blobs = torch.zeros((D, H, W), device="cuda")
    ax = [torch.arange(e, device="cuda", dtype=torch.float32) for e in dhw]
    for b in range(8):
        sig = (8.0 + 24.0 * par[b, 0]) * max(dhw) / 256.0
        amp = (0.2 + 0.6 * par[b, 1]) * torch.sign(par[b, 2] - 0.5)
        gz, gy, gx = (torch.exp(-(ax[i] - par[b, 3 + i] * dhw[i]) ** 2 / (2.0 * sig * sig)) for i in range(3))
        blobs += amp * gz[:, None, None] * gy[None, :, None] * gx[None, None, :]
    return (noise + blobs[None, :, :, :, None]).clamp_(-1.0, 1.0), blobs


def _dhw(case):
    return case["d"], case["h"], case["w"]


def _grid(case):
    return case["gd"], case["gh"], case["gw"]


def prepare(case, seed):
    return (_prepare_block if case["kind"] == "block" else _prepare_net)(case, _generator(seed))


def _prepare_block(case, gen):
    n, dhw, ch = case["n"], _dhw(case), _channels(case)
    dt = sp3d.SP_F32 if case["dtype"] == "f32" else sp3d.SP_BF16
    tdt = sp3d.torch_dtype(dt)
    g = sp3d.Geom(n, dhw, _grid(case))
    train = case["steps"] == "all"
    st = dict(case=case, g=g, dt=dt, ch=ch, w=[], layers=[])
    st["x"] = _ct(gen, n, dhw, 1)[0].to(tdt) if ch[0] == 1 else _normal(gen, (n,) + dhw + (ch[0],), tdt)
    for ci, co in zip(ch, ch[1:]):
        st["w"].append(_normal(gen, (3, 3, 3, ci, co), tdt, math.sqrt(2.0 / (27 * ci))))
    st["P"] = [sp3d.alloc_padded(g, c, dt) for c in ch]                 # layer inputs and the output, margins zero
    st["y"] = torch.empty((n,) + dhw + (ch[-1],), dtype=tdt, device="cuda")
    if train:
        st["dy"] = _normal(gen, (n,) + dhw + (ch[-1],), tdt)
        st["Pd"] = [sp3d.alloc_padded(g, c, dt) for c in ch]            # gradients with respect to them
        st["dx"] = None if _image(ch) else torch.empty((n,) + dhw + (ch[0],), dtype=tdt, device="cuda")
        st["dw"] = [torch.empty((3, 3, 3, ci, co), dtype=torch.float32, device="cuda") for ci, co in zip(ch, ch[1:])]
        st["db"] = [torch.empty((co,), dtype=torch.float32, device="cuda") for co in ch[1:]]
    if case["exchange"] == "messages":
        st["M"] = [sp3d.alloc_msg(g, c, dt) for c in ch]
    gg, nbytes = g.with_opts(sp3d.SP_HALO_GATHER), 16
    for ci, co in zip(ch, ch[1:]):
        can = {op: case["exchange"] == "gather" and sp3d.sp_gather_supported(op, g, ci, co, dt)
               for op in (sp3d.SP_OP_FWD, sp3d.SP_OP_DGRAD, sp3d.SP_OP_WGRAD)}
        gx = can[sp3d.SP_OP_FWD] and (can[sp3d.SP_OP_WGRAD] or not train)
        gz = can[sp3d.SP_OP_DGRAD]
        st["layers"].append((ci, co, gg if gx else g, gg if gz else g))
        nbytes = max([nbytes] + [sp3d.sp_workspace_bytes(op, g, ci, co, dt) for op in can])
    st["gb"] = g.with_opts(KEEP)
    st["ws"] = sp3d.alloc_ws(nbytes)
    return st


def _prepare_net(case, gen):
    n, dhw, ch = case["n"], _dhw(case), _channels(case)
    x, blobs = _ct(gen, n, dhw, case["in_ch"])
    nd, w = 2 if case["flat"] else 3, {}
    for name, shape in unet.layer_plan(ch, case["in_ch"], case["classes"], case["convs"], flat=case["flat"]):
        # Random weights with a positive mean, scaled to keep the activations' size from layer to layer: one ReLU in nine
        # is off.  With zero-mean He weights half of them are, and so many of those by a rounding's width that the
        # gradients of two correct implementations differ by 5 to 8 % at the coarse levels (measured: hidden channels
        # permuted), which would leave nothing to compare.
        fan = math.prod(shape[:nd]) * shape[nd] if name[:2] != "up" else shape[nd]
        mean, std = (0.0, 1.0) if name == "head" else (0.955 / fan, 0.647)
        w[name] = _normal(gen, shape, torch.bfloat16, std / math.sqrt(fan), mean)
    grids = None
    if case["coarse"]:
        coarse = tuple(int(v) for v in case["coarse"].split(","))
        grids = [_grid(case) if i < 3 else coarse for i in range(len(ch))]
    net = unet.UNet(n, dhw, _grid(case), w, ch, case["in_ch"], case["classes"], convs=case["convs"], flat=case["flat"],
                    gather=case["gather"], grids=grids, bits=case["bits"])
    labels = (blobs > 0.1).float() + (blobs > 0.4).float()              # background, organ, lesion
    labels = labels[None, :, :, :, None].expand(n, -1, -1, -1, -1).contiguous().to(torch.bfloat16)
    return dict(case=case, net=net, x=x.to(torch.bfloat16), labels=labels)


# ---- one pass ---------------------------------------------------------------------------------------------------------

def run(state):
    return (_run_block if state["case"]["kind"] == "block" else _run_net)(state)


def _margins(st, P, i):
    """margins of the padded tensor P, which has the channels of layer input i"""
    if "M" in st:
        sp3d.halo_pack(P, st["M"][i], st["gb"], st["ch"][i], st["dt"])
        sp3d.halo_unpack(P, st["M"][i], st["gb"], st["ch"][i], st["dt"])
    else:
        sp3d.sp_halo_exchange(P, st["gb"], st["ch"][i], st["dt"])


def _run_block(st):
    g, dt, ch, P, ws, case = st["g"], st["dt"], st["ch"], st["P"], st["ws"], st["case"]
    last = len(ch) - 2
    sp3d.sp_partition(st["x"], P[0], g, ch[0], dt)
    for i, (ci, co, gx, _) in enumerate(st["layers"]):
        if gx is g:
            _margins(st, P[i], i)
        relu = i < last or case["relu_last"]
        sp3d.conv3d_fwd(P[i], st["w"][i], None, P[i + 1], gx, ci, co, dt, sp3d.SP_FLAG_RELU if relu else 0, ws)
    sp3d.sp_unpartition(P[-1], st["y"], g, ch[-1], dt)
    if case["steps"] != "all":
        return {"y": st["y"]}
    Pd = st["Pd"]
    sp3d.sp_partition(st["dy"], Pd[-1], g, ch[-1], dt)
    if case["relu_last"]:
        sp3d.sp_relu_bwd(Pd[-1], P[-1], Pd[-1], g, ch[-1], dt)
    for i in range(last, -1, -1):
        ci, co, gx, gz = st["layers"][i]
        sp3d.conv3d_wgrad(P[i], Pd[i + 1], st["dw"][i], st["db"][i], gx, ci, co, dt, ws)
        if i == 0 and _image(ch):
            break
        if gz is g:
            _margins(st, Pd[i + 1], i + 1)
        if i:
            sp3d.conv3d_dgrad_relu(Pd[i + 1], st["w"][i], P[i], Pd[i], gz, ci, co, dt, ws)
        else:
            sp3d.conv3d_dgrad(Pd[i + 1], st["w"][i], Pd[i], gz, ci, co, dt, ws)
    if st["dx"] is not None:
        sp3d.sp_unpartition(Pd[0], st["dx"], g, ch[0], dt)
    return {"y": st["y"], "dx": st["dx"], "dw": st["dw"], "db": st["db"]}


def _run_net(st):
    net = st["net"]
    logits = net.forward(st["x"])
    if st["case"]["steps"] != "all":
        return {"logits": logits}
    loss = net.loss(st["labels"])
    grads, _ = net.backward(None, input_grad=False)
    return {"logits": logits, "loss": loss, "grads": grads}
