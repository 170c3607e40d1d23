"""Performance cases of the cache-aware inference path: what a program built on this package has it do.

Three kinds, all through the public entry points of ``paper_1712_01670_amd.binding``:

* ``clip``   ``StackRunner.step`` over ten frames of every stream: one frame computed in full, then nine that reuse the
             previous frame's feature maps.  Ten is the cache's expiry in deployment, so a clip is the steady state of a
             running service, and ten frames follow each other without a wait as they do there.
* ``match``  ``dc_match_blocks_opt`` alone: block matching between two frames of every stream.
* ``layer``  ``dc_cached_conv_layer`` alone: one convolution that takes part of its output from the previous frame's.

The frames are panning textured backgrounds under rigid rectangles of noise that move on their own (camera motion and
moving objects); stacks and frame sizes are those of ``synth.py``, the benchmark and the reuse sweep.

``plan`` of a clip says how a user runs the stack: ``torus`` (planned on the GPU, exact reuse maps, convolution outputs
kept in place: the benchmark's mode, for stacks that qualify), ``maps`` (planned on the GPU, exact reuse maps, shifted
copies: every stack) or ``host`` (``StackRunner``'s defaults: rectangles planned on the host).
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1712_01670_amd import binding, synth

FRAMES = 10        # frames of a clip: the cache expires after that many
DEVICE = "cuda:0"

STACKS = {"tiny": synth.tiny_net, "dave": synth.dave_orig, "vgg16": synth.vgg16, "resnet50": synth.resnet50_trunk,
          "darknet19": synth.darknet19, "alexnet": synth.alexnet, "googlenet": synth.googlenet}


def _clip(name, net, height, width, streams, dtype, plan, search="es", k_skip=1, block=16, moving=0.09, pan=3):
    return dict(name=name, kind="clip", net=net, height=height, width=width, streams=streams, dtype=dtype, plan=plan,
                search=search, k_skip=k_skip, block=block, radius=block, moving=moving, pan=pan)


def listed():
    return [
        # the smallest call: three convolutions on a 64x64 frame with the package's default settings; launches and the
        # host's share are everything
        _clip("tiny 64 f32 x1", "tiny", 64, 64, 1, "f32", "host", block=8),
        # one camera, single precision: the paper's own setting (one video, a VGG-style stack)
        _clip("vgg16 224 f32 x1", "vgg16", 224, 224, 1, "f32", "torus"),
        # one camera in bf16 through a residual network: many short layers, latency again
        _clip("resnet50 224 bf16 x1", "resnet50", 224, 224, 1, "bf16", "maps"),
        # one camera through a detection stack at its usual 416x416
        _clip("darknet19 416 bf16 x1", "darknet19", 416, 416, 1, "bf16", "torus"),
        # a camera hub: five streams of a size that divides by nothing, the default host-planned rectangles
        _clip("vgg16 187x250 bf16 x5", "vgg16", 187, 250, 5, "bf16", "host"),
        # batched serving: 16 streams of each of the larger stacks ...
        _clip("resnet50 224 bf16 x16", "resnet50", 224, 224, 16, "bf16", "maps"),
        _clip("googlenet 224 bf16 x16", "googlenet", 224, 224, 16, "bf16", "maps"),
        # ... with the diamond search and k-skip of the paper on the larger frames
        _clip("darknet19 416 bf16 x16", "darknet19", 416, 416, 16, "bf16", "torus", search="ds", k_skip=2),
        # 64 streams with fully-connected layers at the end
        _clip("alexnet 227 bf16 x64", "alexnet", 227, 227, 64, "bf16", "maps"),
        # the throughput configuration of the benchmark, the largest
        _clip("vgg16 224 bf16 x64", "vgg16", 224, 224, 64, "bf16", "torus"),
        # the matching alone, as a caller runs it that only wants the motion of 16 streams
        dict(name="match 416 x16", kind="match", height=416, width=416, channels=3, streams=16, search="es", k_skip=1,
             block=16, radius=16, moving=0.09, pan=3),
        # one convolution of a caller that runs its own layer loop, two fifths of its output reused
        dict(name="layer 3x3 256 56 bf16 x8", kind="layer", k=3, s=1, p=1, cin=256, cout=256, height=56, width=56, streams=8,
             dtype="bf16", reuse=0.4),
    ]


def _log_uniform(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


# frame edges a stack is run on in earnest (smallest, largest); equal: the stack has one frame size
_EDGES = {"tiny": ((48, 128), (48, 128)), "dave": ((66, 66), (200, 200)), "vgg16": ((96, 360), (96, 480)),
          "resnet50": ((128, 320), (128, 320)), "darknet19": ((224, 608), (224, 608)), "alexnet": ((227, 227), (227, 227)),
          "googlenet": ((224, 224), (224, 224))}


def _cost(case):
    """Rough time of a pass, for the bound on drawn cases: convolutions at 0.45 of the matrix units' peaks (fp32 runs at a
    sixteenth of bf16), feature maps through memory, and a launch per layer."""
    flops = _conv_flops(case, full=True)
    peak = 2.5e15 if case["dtype"] == "bf16" else 157e12
    maps, launches = 0.0, 1
    if case["kind"] == "clip":
        shapes = synth.tensor_shapes(_stack(case), case["height"], case["width"], 3)
        maps = FRAMES * case["streams"] * sum(h * w * c for h, w, c in shapes) * (2 if case["dtype"] == "bf16" else 4)
        launches = FRAMES * len(shapes)
    return flops / peak / 0.45 + 1.5 * maps / 5e12 + 5e-6 * launches


def draw(rng):
    """A case of the same ranges: any stack, any frame size and number of streams it is run with, both data types."""
    kind = rng.choice(["clip"] * 6 + ["match", "layer"])
    if kind == "match":
        block = rng.choice([8, 16, 16])
        return dict(kind="match", height=_log_uniform(rng, 64, 640), width=_log_uniform(rng, 64, 640), channels=3,
                    streams=_log_uniform(rng, 1, 32), search=rng.choice(["es", "es", "ds"]), k_skip=rng.choice([1, 1, 2]),
                    block=block, radius=block, moving=round(rng.uniform(0.0, 0.4), 3), pan=rng.choice([0, 1, 2, 3, 3]))
    limit = 0.6 * _cost(listed()[9])
    if kind == "layer":
        k = rng.choice([1, 3, 3, 3, 5])
        case = dict(kind="layer", k=k, s=rng.choice([1, 1, 1, 2]), p=k // 2, cin=rng.choice([32, 48, 64, 96, 128, 256, 384, 512]),
                    cout=rng.choice([32, 64, 96, 128, 256, 384, 512]), height=_log_uniform(rng, 7, 112),
                    width=_log_uniform(rng, 7, 112), streams=_log_uniform(rng, 1, 32), dtype=rng.choice(["bf16", "bf16", "f32"]),
                    reuse=round(rng.uniform(0.0, 0.8), 3))
        while _cost(case) > limit:
            case["streams"] = max(1, case["streams"] // 2)
        return case
    net = rng.choice(["tiny", "dave", "vgg16", "vgg16", "resnet50", "darknet19", "darknet19", "alexnet", "googlenet"])
    (h0, h1), (w0, w1) = _EDGES[net]
    height, width = _log_uniform(rng, h0, h1), _log_uniform(rng, w0, w1)
    dtype = rng.choice(["bf16", "bf16", "f32"])
    plans = ["torus", "torus", "torus", "maps", "host"] if net in ("vgg16", "darknet19") else ["maps", "maps", "host"]
    search = rng.choice(["es", "es", "ds"])
    case = dict(kind="clip", net=net, height=height, width=width, streams=_log_uniform(rng, 1, 64), dtype=dtype,
                plan=rng.choice(plans), search=search, k_skip=rng.choice([1, 2]) if search == "ds" else 1,
                block=8 if net == "tiny" else 16, radius=8 if net == "tiny" else 16,
                moving=round(rng.uniform(0.0, 0.4), 3), pan=rng.choice([0, 1, 2, 3, 3]))
    while _cost(case) > limit and case["streams"] > 1:
        case["streams"] //= 2
    return case


# --------------------------------------------------------------------------- #
# inputs                                                                      #
# --------------------------------------------------------------------------- #
def _tracks(case, rng, frames):
    """Geometry of one stream's video: view origins [frames] and moving rectangles [frames][(x, y, w, h)]."""
    H, W, pan = case["height"], case["width"], case["pan"]
    dx, dy = [(1, 0), (1, 1), (0, 1), (-1, 1), (-1, 0), (-1, -1), (0, -1), (1, -1)][rng.integers(8)]
    speed = int(rng.integers(1, pan + 1)) if pan else 0
    views = [(f * dx * speed, f * dy * speed) for f in range(frames)]
    boxes = [[] for _ in range(frames)]
    for aspect in (1.0, 2.0):                        # a square and an upright rectangle, half the moving area each
        area = case["moving"] * H * W / 2
        w = min(int(round(math.sqrt(area / aspect))), W)
        h = min(int(round(math.sqrt(area * aspect))), H)
        if w < 1 or h < 1:
            continue
        x, y = int(rng.integers(0, W - w + 1)), int(rng.integers(0, H - h + 1))
        ux, uy = (int(v) for v in rng.choice([-6, -5, -4, 4, 5, 6], 2))
        for f in range(frames):
            if f:
                x, y = x + ux, y + uy
                ux = -ux if x < 0 or x + w > W else ux
                uy = -uy if y < 0 or y + h > H else uy
                x, y = min(max(x, 0), W - w), min(max(y, 0), H - h)
            boxes[f].append((x, y, w, h))
    return views, boxes


def _video(case, seed, frames):
    """uint8 [frames][streams][H][W][3] on the GPU: value noise (five octaves) under moving rectangles of noise."""
    H, W, n, C = case["height"], case["width"], case["streams"], 3
    margin = case["pan"] * frames
    gen = torch.Generator(DEVICE)
    gen.manual_seed(seed)
    Hc, Wc = H + 2 * margin, W + 2 * margin
    canvas = torch.zeros((n, Hc, Wc, C), device=DEVICE)
    total, amp = 0.0, 1.0
    for lattice in (64, 32, 16, 8, 4):
        grid = torch.rand((n, Hc // lattice + 2, Wc // lattice + 2, C), generator=gen, device=DEVICE)

        def axis(size):
            g = torch.arange(size, device=DEVICE, dtype=torch.float32) / lattice
            i = g.floor().long()
            t = g - i
            return i, t * t * (3.0 - 2.0 * t)
        iy, ty = axis(Hc)
        ix, tx = axis(Wc)
        rows = torch.lerp(grid[:, iy], grid[:, iy + 1], ty[None, :, None, None])
        canvas += amp * torch.lerp(rows[:, :, ix], rows[:, :, ix + 1], tx[None, None, :, None])
        total += amp
        amp *= 0.5
    canvas = (canvas * (255.0 / total)).round_().clamp_(0, 255).to(torch.uint8)
    rng = np.random.default_rng(seed)
    out = torch.empty((frames, n, H, W, C), dtype=torch.uint8, device=DEVICE)
    noise = torch.randint(0, 256, (n, H, W, C), generator=gen, device=DEVICE, dtype=torch.uint8)
    for s in range(n):
        views, boxes = _tracks(case, rng, frames)
        for f in range(frames):
            ox, oy = margin + views[f][0], margin + views[f][1]
            out[f, s] = canvas[s, oy:oy + H, ox:ox + W]
            for (x, y, w, h) in boxes[f]:            # rigid: the texture moves with its rectangle
                out[f, s, y:y + h, x:x + w] = noise[s, :h, :w]
    return out


_weights = {}      # a model's weights are the same for every video: drawn once per process


def _stack(case):
    H, W = case["height"], case["width"]
    return synth.resolve_global_pooling(STACKS[case["net"]](), H, W, 3)


def prepare(case, seed):
    torch.cuda.set_device(torch.device(DEVICE))
    state = {"case": case}
    if case["kind"] == "layer":
        gen = torch.Generator(DEVICE)
        gen.manual_seed(seed)
        dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
        n, H, W, k, cin, cout = (case[f] for f in ("streams", "height", "width", "k", "cin", "cout"))
        layer = dict(type=synth.CONV, k=k, s=case["s"], p=case["p"], cin=cin, cout=cout, relu=1, in0=0, in1=-1)
        ho, wo, _ = synth.tensor_shapes([layer], H, W, cin)[1]
        normal = lambda *shape: torch.randn(shape, generator=gen, device=DEVICE)
        state["x"] = normal(n, H, W, cin).clamp_(min=0).to(dt)                       # the layer before ended in a ReLU
        state["w"] = (normal(cout, k, k, cin) * math.sqrt(2.0 / (cin * k * k))).to(dt)
        state["b"] = normal(cout) * 0.05
        state["prev"] = normal(n, ho, wo, cout).clamp_(min=0).to(dt)
        state["packed"] = binding.dc_pack_conv_weights(layer, state["w"])
        state["layer"] = layer
        state["regions"] = [_rects(case, np.random.default_rng((seed, s)), ho, wo) for s in range(n)]
        return state
    if case["kind"] == "match":
        video = _video(case, seed, 2)
        state["prev"], state["cur"] = video[0], video[1]
        state["bound"] = synth.max_block_ssd(case["block"], 3)
        return state
    layers = _stack(case)
    key = (case["net"], case["height"], case["width"])
    if key not in _weights:
        _weights.clear()
        _weights[key] = synth.he_weights(layers, 1, residual_scale=0.5 if case["net"] == "resnet50" else 1.0,
                                         input_shape=(case["height"], case["width"], 3))
    ws, bs = _weights[key]
    state["video"] = _video(case, seed, FRAMES)
    state["runner"] = binding.StackRunner(
        layers, ws, bs, case["streams"], case["height"], case["width"], 3, block=case["block"], radius=case["radius"],
        dtype=binding.DC_BF16 if case["dtype"] == "bf16" else binding.DC_F32, expiry=FRAMES, match_method=_method(case),
        k_skip=case["k_skip"], device_plan=case["plan"] != "host", exact_masks=case["plan"] != "host",
        torus=case["plan"] == "torus")
    return state


def _method(case):
    return binding.DC_MATCH_DIAMOND if case["search"] == "ds" else binding.DC_MATCH_EXHAUSTIVE


def _rects(case, rng, ho, wo):
    """Two reusable rectangles side by side (rects, source offset) that cover about `reuse` of the map."""
    dx, dy = int(rng.integers(-1, 2)), int(rng.integers(-1, 2))
    h = int((ho - 2) * math.sqrt(case["reuse"]))
    w = int((wo - 2) * math.sqrt(case["reuse"])) // 2
    if h < 1 or w < 1:
        return np.zeros((0, 4), np.int32), (dx, dy)
    y, x = int(rng.integers(1, ho - h)), int(rng.integers(1, wo - 2 * w))
    return np.array([[x, y, w, h], [x + w, y, w, h]], np.int32), (dx, dy)


# --------------------------------------------------------------------------- #
# one pass                                                                    #
# --------------------------------------------------------------------------- #
def run(state):
    case = state["case"]
    if case["kind"] == "layer":
        return binding.dc_cached_conv_layer(state["layer"], state["x"], state["w"], state["b"], state["prev"],
                                            state["regions"], packed=state["packed"])
    if case["kind"] == "match":
        return binding.dc_match_blocks_opt(state["cur"], state["prev"], case["block"], case["radius"], state["bound"],
                                           _method(case), case["k_skip"])
    runner, video = state["runner"], state["video"]
    for f in range(FRAMES):
        tensors = runner.step(video[f])
    # what the application takes from the last frame: the stack's output and the last convolution's map (the cache that the
    # next frame would reuse), and the motion of every block
    last_conv = max(i for i, L in enumerate(runner.layers) if L["type"] == synth.CONV) + 1
    out = {"out": runner.read_tensor(len(runner.layers), tensors), "mv": runner.mv, "gmv": runner.gmv, "mask": runner.mask}
    if last_conv < len(runner.layers):
        out["map"] = runner.read_tensor(last_conv, tensors)
    return out


# --------------------------------------------------------------------------- #
# what a pass cannot do without                                               #
# --------------------------------------------------------------------------- #
def _match_ops(case):
    """Integer operations of the exhaustive search; the diamond search visits about 20 of the candidates."""
    blocks = (case["height"] // case["block"]) * (case["width"] // case["block"]) * case["streams"]
    candidates = (2 * case["radius"] + 1) ** 2 if case["search"] == "es" else 20
    return 2.0 * blocks / case["k_skip"] ** 2 * candidates * case["block"] ** 2 * 3


def _eroded(mask, k, s, p):
    """Outputs whose k x k window lies inside the set (windows that touch the padding do not)."""
    (kh, kw), (ph, pw) = k, p
    m = np.pad(mask, ((ph, ph), (pw, pw)))
    rows = np.lib.stride_tricks.sliding_window_view(m, kh, axis=0).all(-1)
    return np.lib.stride_tricks.sliding_window_view(rows, kw, axis=1).all(-1)[::s, ::s]


def _conv_flops(case, full=False):
    """Multiply-adds x 2 of the output pixels that have to be computed: all of a full frame's, and on the other frames
    those outside the reuse maps that follow from the video's geometry (one stream stands for all)."""
    if case["kind"] == "layer":
        layer = dict(type=synth.CONV, k=case["k"], s=case["s"], p=case["p"], cin=case["cin"], cout=case["cout"], in0=0, in1=-1)
        ho, wo, _ = synth.tensor_shapes([layer], case["height"], case["width"], case["cin"])[1]
        rects, _ = _rects(case, np.random.default_rng(0), ho, wo)
        px = ho * wo - (0 if full else int((rects[:, 2] * rects[:, 3]).sum()))
        return 2.0 * case["streams"] * px * case["k"] ** 2 * case["cin"] * case["cout"]
    layers = _stack(case)
    H, W, B = case["height"], case["width"], case["block"]
    shapes = synth.tensor_shapes(layers, H, W, 3)
    views, boxes = _tracks(case, np.random.default_rng(0), 2)
    mask = np.zeros((H, W), bool)
    for by in range(0, H - B + 1, B):
        for bx in range(0, W - B + 1, B):
            sx, sy = bx + views[1][0], by + views[1][1]            # where the block lay one frame ago
            fits = 0 <= sx <= W - B and 0 <= sy <= H - B
            clear = all(bx >= x + w or bx + B <= x or by >= y + h or by + B <= y for (x, y, w, h) in boxes[1]) and \
                all(sx >= x + w or sx + B <= x or sy >= y + h or sy + B <= y for (x, y, w, h) in boxes[0])
            mask[by:by + B, bx:bx + B] = fits and clear
    masks, flops_full, flops_cached = [mask], 0.0, 0.0
    for i, L in enumerate(layers):
        src = masks[L["in0"]]
        if full:
            out = src
        elif L["type"] in (synth.CONV, synth.MAXPOOL, synth.AVGPOOL):
            kh, kw, ph, pw, _ = synth.conv_geometry(L)
            out = _eroded(src, (kh, kw), L["s"], (ph, pw))
        elif L["type"] in (synth.ADD, synth.CONCAT):
            out = np.logical_and.reduce([masks[L[f]] for f in ("in0", "in1", "in2", "in3") if L.get(f, -1) >= 0])
        elif L["type"] in (synth.FC, synth.SOFTMAX):
            out = np.zeros((1, 1), bool)
        else:
            out = src
        masks.append(out)
        ho, wo, co = shapes[i + 1]
        if L["type"] == synth.CONV:
            per_px = 2.0 * synth.conv_geometry(L)[0] * synth.conv_geometry(L)[1] * L["cin"] * L["cout"]
            flops_full += per_px * ho * wo
            flops_cached += per_px * (ho * wo if full else ho * wo - int(out.sum()))
        elif L["type"] == synth.FC:
            flops = 2.0 * co * int(np.prod(shapes[L["in0"]]))
            flops_full += flops
            flops_cached += flops
    return case["streams"] * (flops_full + (FRAMES - 1) * flops_cached)


def work(case):
    n = case["streams"]
    es = 2 if case.get("dtype") == "bf16" else 4
    if case["kind"] == "match":
        blocks = n * (case["height"] // case["block"]) * (case["width"] // case["block"])
        return {"bytes": 2.0 * n * case["height"] * case["width"] * 3 + 9.0 * blocks, "flops": _match_ops(case)}
    if case["kind"] == "layer":
        layer = dict(type=synth.CONV, k=case["k"], s=case["s"], p=case["p"], cin=case["cin"], cout=case["cout"], in0=0, in1=-1)
        ho, wo, co = synth.tensor_shapes([layer], case["height"], case["width"], case["cin"])[1]
        values = n * (case["height"] * case["width"] * case["cin"] + (1 + case["reuse"]) * ho * wo * co) + \
            case["k"] ** 2 * case["cin"] * co
        return {"bytes": float(es * values), "flops": _conv_flops(case)}
    layers = _stack(case)
    shapes = synth.tensor_shapes(layers, case["height"], case["width"], 3)
    weights = sum(synth.conv_geometry(L)[0] * synth.conv_geometry(L)[1] * L["cin"] * L["cout"] for L in layers if L["type"] == synth.CONV) + \
        sum(int(np.prod(shapes[L["in0"]])) * L["cout"] for L in layers if L["type"] == synth.FC)
    out = int(np.prod(shapes[-1]))
    return {"bytes": FRAMES * n * (3.0 * case["height"] * case["width"] + es * out) + es * float(weights), "flops": _conv_flops(case)}


def tolerance(case):
    """Integer results (vectors, masks) are the same; features differ by the order of fp32 sums, rounded to the storage
    type after every layer."""
    if case["kind"] == "match":
        return "exact"
    return {"rel": 1e-2} if case["dtype"] == "bf16" else {"rel": 1e-5}
