"""The work this library is measured on: sparse video inference through `Net`, and mask compaction through `Context`.

A pass of a network case is ONE frame of every camera stream (`Net.step`, or `Net.init` for the dense first frame),
with the frames resident on the GPU, and returns the network's dense output.  The streams show a textured static
background, sensor noise and moving objects; a case keeps a short clip that is played forwards and backwards, so every
pass sees a frame that differs from the one before it.
"""
import math
import random

import numpy as np
import torch
import torch.nn.functional as F

import paper_2203_03996_amd as pkg

CLIP = 5                                            # frames of a clip: played 1 2 3 4 3 2 1 0 1 2 ...
ORDER = list(range(1, CLIP)) + list(range(CLIP - 2, -1, -1))
NP_TYPE = {"f16": np.float16, "f32": np.float32}
TORCH_TYPE = {"f16": torch.float16, "f32": torch.float32}
SIZE = {"f16": 2, "f32": 4}


# ---- topologies (node tables as `Net` takes them) -----------------------------------------------------------------
class _Nodes(list):
    def __init__(self, eps0, eps, f="relu"):
        super().__init__()
        self.eps, self.f = eps, f
        self.append({"kind": "deltagen", "in": [], "eps": eps0})

    def add_node(self, kind, *inputs, **attributes):
        self.append({"kind": kind, "in": list(inputs), **attributes})
        return len(self) - 1

    def conv(self, x, k, s, cin, cout, depthwise=False, gain=1.0):
        return self.add_node("conv", x, k=k, stride=s, pad=k // 2, cin=cin, cout=cout, depthwise=depthwise, gain=gain)

    def act(self, x):
        return self.add_node("act", x, f=self.f, eps=self.eps)

    def conv_act(self, *a, **kw):
        return self.act(self.conv(*a, **kw))


RESIDUAL = 0.3                                      # gain of a residual branch: activations keep their scale with depth


def _bottleneck(b, x, cin, mid, cout, s, project):
    y = b.conv_act(x, 1, 1, cin, mid)
    y = b.conv_act(y, 3, s, mid, mid)
    y = b.conv(y, 1, 1, mid, cout, gain=RESIDUAL)
    if project:
        x = b.conv(x, 1, s, cin, cout)
    return b.act(b.add_node("add", y, x))


def nodes_of(case):
    """The topology of a case; `eps0` is the threshold of the input layer, `eps` of every activation."""
    net, c = case["net"], case["c"]
    b = _Nodes(case["eps0"], case["eps"], "relu6" if net == "mobilenet" else "relu")
    if net == "conv":                               # one convolution, with or without the activation behind it
        x = b.conv(0, case["k"], case["stride"], c, case["cout"])
        x = b.act(x) if case["act"] else x
    elif net == "block":                            # ResNet bottleneck with a projection shortcut
        x = _bottleneck(b, 0, c, case["mid"], case["cout"], 1, True)
    elif net == "mobilenet":                        # inverted residuals, expansion 6, depthwise 3x3
        x = b.conv_act(0, 3, 2, c, 32)
        for cin, cout, s in ((32, 32, 1), (32, 48, 2), (48, 48, 1), (48, 64, 2), (64, 96, 1), (96, 160, 2), (160, 160, 1)):
            y = b.conv_act(x, 1, 1, cin, 6 * cin)
            y = b.conv_act(y, 3, s, 6 * cin, 6 * cin, depthwise=True)
            y = b.conv(y, 1, 1, 6 * cin, cout, gain=RESIDUAL if s == 1 and cin == cout else 1.0)
            x = b.add_node("add", x, y) if s == 1 and cin == cout else y
    elif net == "resnet":                           # 7x7 stem, max-pool, four stages of bottlenecks
        x = b.conv_act(0, 7, 2, c, 64)
        x = b.add_node("maxpool", x, k=3, stride=2, pad=1)
        cin = 64
        for stage, blocks in enumerate((3, 4, 6, 3)):
            mid = 64 << stage
            for i in range(blocks):
                x = _bottleneck(b, x, cin, mid, 4 * mid, 2 if i == 0 and stage else 1, i == 0)
                cin = 4 * mid
    elif net == "hrnet":                            # parallel branches at 1/4 .. 1/32, every one fused into every other
        widths = (32, 64, 128, 256)
        x = b.conv_act(b.conv_act(0, 3, 2, c, 64), 3, 2, 64, 64)
        branch = [b.conv_act(x, 3, 1, 64, 32), b.conv_act(x, 3, 2, 64, 64)]
        for _ in range(3):
            for i, x in enumerate(branch):
                y = b.conv(b.conv_act(x, 3, 1, widths[i], widths[i]), 3, 1, widths[i], widths[i], gain=RESIDUAL)
                branch[i] = b.act(b.add_node("add", y, x))
            fused = []
            for i in range(len(branch)):
                total = None
                for j, t in enumerate(branch):
                    if j > i:
                        t = b.add_node("upsample", b.conv(t, 1, 1, widths[j], widths[i], gain=RESIDUAL), factor=2 ** (j - i))
                    for step in range(i - j):
                        last = step == i - j - 1
                        t = b.conv(t, 3, 2, widths[j], widths[i] if last else widths[j], gain=RESIDUAL if last else 1.0)
                        t = t if last else b.act(t)
                    total = t if total is None else b.add_node("add", total, t)
                fused.append(b.act(total))
            branch = fused
            if len(branch) < 4:
                branch.append(b.conv_act(branch[-1], 3, 2, widths[len(branch) - 1], widths[len(branch)]))
        x = branch[0]
        for j in range(1, 4):
            x = b.add_node("add", x, b.add_node("upsample", b.conv(branch[j], 1, 1, widths[j], 32), factor=2 ** j))
        x = b.conv(b.act(x), 1, 1, 32, 16)
    elif net == "decoder":                          # a coarser branch brought back up and joined with the input
        x = b.conv_act(0, 3, 2, c, case["mid"])
        x = b.add_node("upsample_bilinear", b.conv(x, 1, 1, case["mid"], c), factor=2)
        x = b.add_node("concat", x, 0)
        x = b.conv_act(x, 5, 1, 2 * c, case["cout"])
    else:
        raise ValueError(net)
    b.add_node("accum", x)
    return list(b)


def _shapes(case, nodes):
    got = [(case["h"], case["w"], case["c"])]
    for nd in nodes[1:]:
        h, w, c = got[nd["in"][0]]
        if nd["kind"] in ("conv", "maxpool"):
            h, w = ((v + 2 * nd["pad"] - nd["k"]) // nd["stride"] + 1 for v in (h, w))
            c = nd.get("cout", c)
        elif nd["kind"].startswith("upsample"):
            h, w = h * nd["factor"], w * nd["factor"]
        elif nd["kind"] == "concat":
            c += got[nd["in"][1]][2]
        got.append((h, w, c))
    return got


# ---- inputs ----------------------------------------------------------------------------------------------------------
def _weights(case, nodes, seed):
    """He-normal weights and small biases, rounded to the storage type, by node index."""
    rng = np.random.default_rng(seed)
    t = NP_TYPE[case["dtype"]]
    made = {}
    for i, nd in enumerate(nodes):
        if nd["kind"] == "conv":
            k, cout = nd["k"], nd["cout"]
            shape, fan = ((k, k, cout), k * k) if nd["depthwise"] else ((k, k, nd["cin"], cout), k * k * nd["cin"])
            made[i] = ((rng.standard_normal(shape, dtype=np.float32) * np.float32(nd["gain"] * math.sqrt(2.0 / fan))).astype(t),
                       (0.01 * rng.standard_normal(cout)).astype(t))
    return made


def _clip(case, seed):
    """The frames of a clip, [streams, h, w, c] each.  "video": moving textured objects over a smooth background, with
    sensor noise everywhere; "random": new values at uniformly random pixels of every frame (no spatial structure)."""
    n, h, w, c = case["streams"], case["h"], case["w"], case["c"]
    g = torch.Generator(device="cuda").manual_seed(seed)
    randn = lambda *s: torch.randn(s, generator=g, device="cuda")  # noqa: E731
    coarse = randn(n, c, -(-h // 8) + 1, -(-w // 8) + 1)
    base = F.interpolate(coarse, size=(h, w), mode="bilinear", align_corners=True).permute(0, 2, 3, 1).contiguous()
    base /= base.std()
    frames = []
    if case["video"] == "random":
        for _ in range(CLIP):
            new = torch.rand((n, h, w, 1), generator=g, device="cuda") < case["changed"]
            base = torch.where(new, randn(n, h, w, c), base)
            frames.append(base.to(TORCH_TYPE[case["dtype"]]))
        return frames
    r = random.Random(seed)
    side = max(2, min(h, w) // 10)
    things = [[r.randint(0, h - side), r.randint(0, w - side), r.choice((-3, -2, -1, 1, 2, 3)), r.choice((-3, -2, -1, 1, 2, 3)), s]
              for s in range(n) for _ in range(case["objects"])]
    look = randn(max(1, len(things)), side, side, c) + 1.0
    for _ in range(CLIP):
        frame = base + case["noise"] * randn(n, h, w, c)
        for i, t in enumerate(things):
            frame[t[4], t[0]:t[0] + side, t[1]:t[1] + side] = look[i]
            for axis, end in ((0, h - side), (1, w - side)):
                if not 0 <= t[axis] + t[axis + 2] <= end:
                    t[axis + 2] = -t[axis + 2]
                t[axis] = min(end, max(0, t[axis] + t[axis + 2]))
        frames.append(frame.to(TORCH_TYPE[case["dtype"]]))
    return frames


def _masks(case, seed):
    """Update masks: rectangles that moved, and single noisy pixels."""
    n, h, w = case["streams"], case["h"], case["w"]
    g = torch.Generator(device="cuda").manual_seed(seed)
    mask = torch.rand((n, h, w), generator=g, device="cuda") < case["changed"]
    r = random.Random(seed)
    for s in range(n):
        y, x = r.randint(0, h - 1), r.randint(0, w - 1)
        mask[s, y:y + max(1, h // 5), x:x + max(1, w // 5)] = True
    return mask.to(torch.uint8)


# ---- cases -------------------------------------------------------------------------------------------------------------
def _net(net, dtype, streams, h, w, c, **more):
    case = {"net": net, "dtype": dtype, "streams": streams, "h": h, "w": w, "c": c, "video": "video", "objects": 8,
            "noise": 0.01, "eps0": 0.05, "eps": 0.05, "active": 0.1, "first": False}
    case.update(more)
    return case


def _compact(streams, h, w, k, stride, changed=0.02):
    return {"net": "mask_compact", "streams": streams, "h": h, "w": w, "k": k, "stride": stride, "pad": k // 2, "changed": changed}


def listed():
    return [
        # the smallest network, fp32: launches and latency
        dict(_net("conv", "f32", 1, 64, 64, 32, k=3, stride=1, cout=32, act=True, objects=2), name="conv3x3_relu_f32_1"),
        # one camera through a ResNet bottleneck: the latency of a live stream
        dict(_net("block", "f16", 1, 128, 128, 64, mid=64, cout=256), name="block_1"),
        # 64 cameras batched: throughput, the benchmark's workload
        dict(_net("block", "f16", 64, 128, 128, 64, mid=64, cout=256), name="block_64"),
        # the same block in fp32 on maps whose rows are no multiple of anything
        dict(_net("block", "f32", 8, 117, 93, 64, mid=64, cout=256), name="block_8_f32_ragged"),
        # the dense first frame of 64 cameras (start of a video, and every reset against drift)
        dict(_net("block", "f16", 64, 128, 128, 64, mid=64, cout=256, first=True, active=1.0), name="block_64_first"),
        # whole networks, 8 cameras: depthwise inverted residuals; a deep chain; parallel resolutions
        dict(_net("mobilenet", "f16", 8, 224, 224, 3, eps0=0.06, eps=0.2, active=0.3), name="mobilenet_8"),
        dict(_net("resnet", "f16", 8, 256, 256, 3, eps0=0.06, eps=0.4, active=0.4), name="resnet50_8"),
        dict(_net("resnet", "f16", 8, 256, 256, 3, eps0=0.06, eps=0.4, first=True, active=1.0), name="resnet50_8_first"),
        dict(_net("hrnet", "f16", 8, 384, 288, 3, eps0=0.06, eps=0.2, objects=2), name="hrnet_8"),
        # one wide convolution under updates without spatial structure (the worst case for skipping)
        dict(_net("conv", "f16", 8, 256, 256, 128, k=3, stride=1, cout=128, act=False, video="random", changed=0.1, active=0.6),
             name="conv3x3_128_random_8"),
        # odd channel counts, a 5x5 window, bilinear upsampling and concatenation on small maps
        dict(_net("decoder", "f16", 3, 118, 94, 20, mid=27, cout=24, active=0.15), name="decoder_3_odd"),
        # the list of pixels to visit, from a caller's own mask
        dict(_compact(48, 127, 95, 3, 1), name="mask_compact_48"),
    ]


def _spread(rng, low, high):
    """A whole number between low and high, even over its logarithm."""
    return int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))


def draw(rng):
    kind = rng.choice(("conv", "conv", "block", "block", "mobilenet", "resnet", "hrnet", "decoder", "mask_compact"))
    if kind == "mask_compact":
        return _compact(_spread(rng, 1, 64), rng.randint(17, 200), rng.randint(17, 200), rng.choice((1, 3, 5, 7)), rng.choice((1, 2)),
                        rng.choice((0.005, 0.02, 0.1, 0.5)))
    dtype = "f32" if rng.random() < 0.25 else "f16"
    more = {"first": rng.random() < 0.25, "objects": rng.randint(2, 12)}
    if kind == "block":
        mid = rng.choice((32, 64))
        case = _net(kind, dtype, _spread(rng, 1, 40), rng.randint(40, 128), rng.randint(40, 128), rng.choice((32, 64)), mid=mid,
                    cout=4 * mid, eps=rng.choice((0.05, 0.1)), **more)
    elif kind == "conv":
        k = rng.choice((1, 3, 3, 5, 7))
        if k <= 3 and rng.random() < 0.4:               # any channel counts
            c, cout = rng.randint(3, 40), rng.randint(5, 48)
        else:
            c, cout = 8 * rng.randint(2, 16), 8 * rng.randint(2, 16)
        case = _net(kind, dtype, _spread(rng, 1, 8), rng.randint(30, 200), rng.randint(30, 200), c, k=k, stride=rng.choice((1, 1, 2)),
                    cout=cout, act=rng.random() < 0.7, **more)
        if rng.random() < 0.3:
            case.update(video="random", changed=rng.choice((0.02, 0.1, 0.5)))
    elif kind == "decoder":
        case = _net(kind, "f16", _spread(rng, 1, 8), 2 * rng.randint(20, 90), 2 * rng.randint(20, 90), rng.randint(4, 24),
                    mid=rng.randint(8, 40), cout=rng.randint(8, 32), **more)
    else:
        h, w = rng.randint(96, 224), rng.randint(96, 224)
        if kind == "hrnet":
            h, w = 32 * rng.randint(3, 10), 32 * rng.randint(3, 9)
        case = _net(kind, dtype, _spread(rng, 1, 8), h, w, 3, eps0=0.06, eps=rng.choice((0.1, 0.2, 0.4)), **more)
    usual = {"mobilenet": 0.3, "resnet": 0.4, "hrnet": 0.25}
    case["active"] = 1.0 if case["first"] else case.get("changed", usual.get(kind, 0.1))
    return case


def prepare(case, seed):
    n, h, w = case["streams"], case["h"], case["w"]
    if case["net"] == "mask_compact":
        k, s, p = case["k"], case["stride"], case["pad"]
        oh, ow = (h + 2 * p - k) // s + 1, (w + 2 * p - k) // s + 1
        return {"case": case, "ctx": pkg.Context(n * h * w), "masks": [_masks(case, seed), _masks(case, seed + 1)], "next": 0,
                "mask": torch.zeros((n, oh, ow), dtype=torch.uint8, device="cuda"),
                "idx": torch.zeros(n * oh * ow, dtype=torch.int32, device="cuda"),
                "count": torch.zeros(1, dtype=torch.int32, device="cuda")}
    nodes = nodes_of(case)
    shapes = _shapes(case, nodes)
    ctx = pkg.Context(max(n * a * b for a, b, _ in shapes))
    net = pkg.Net(ctx, {"nodes": nodes, "dtype": case["dtype"], "h": h, "w": w, "c": case["c"]}, _weights(case, nodes, seed), n)
    frames = _clip(case, seed)
    net.init(frames[0])
    kept = {}
    if case["net"] in ("conv", "block", "decoder"):     # the buffers a frame updates: the stored input and every accumulated input
        for i in range(net.num_layers):
            node = net.layer_node(i)
            if nodes[node]["kind"] in ("deltagen", "act"):
                kept["state%d" % node] = net.layer_state(i, 0).view(n, *shapes[node])
    return {"case": case, "ctx": ctx, "net": net, "frames": frames, "kept": kept, "next": 0}


def run(state):
    case, k = state["case"], state["next"]
    state["next"] = k + 1
    if case["net"] == "mask_compact":
        out = {name: state[name] for name in ("mask", "idx", "count")}
        state["ctx"].mask_compact_static(state["masks"][k % 2], out["mask"], out["idx"], out["count"], case["k"], case["stride"], case["pad"])
        return out
    net, frame = state["net"], state["frames"][ORDER[k % len(ORDER)]]
    if case["first"]:
        net.init(frame)
    else:
        net.step(frame)
    return dict(state["kept"], out=net.output().data)


def work(case):
    """A frame is read and compared with the stored one, and at the `active` share of the pixels every accumulated input is
    read and written and the output is written; weights are read once.  (First frame: everything is written.)"""
    n = case["streams"]
    if case["net"] == "mask_compact":
        px = n * case["h"] * case["w"]
        out = px / case["stride"] ** 2
        return {"bytes": px + out + 4 * out * min(1.0, 0.04 + case["changed"] * case["k"] ** 2), "flops": 0}
    nodes, size, active = nodes_of(case), SIZE[case["dtype"]], case["active"]
    shapes = _shapes(case, nodes)
    elems = [n * h * w * c for h, w, c in shapes]
    macs = weights = state = 0
    for i, nd in enumerate(nodes):
        if nd["kind"] == "conv":
            per = nd["k"] ** 2 * (1 if nd["depthwise"] else nd["cin"])
            macs += elems[i] * per
            weights += per * nd["cout"]
        elif nd["kind"] == "act":
            state += elems[i]
    moved = (elems[0] + elems[0] + state + elems[-1]) if case["first"] else 2 * elems[0] + active * (elems[0] + 2 * state + elems[-1])
    return {"bytes": size * (moved + weights), "flops": 2.0 * active * macs}


def tolerance(case):
    """Four times the difference from the same frames in 64 bits (`exact`), which is one rounding per stored value and, in
    fp16, now and then a pixel whose change lies so close to the threshold that the rounding decides it (`max`)."""
    if case["net"] == "mask_compact":
        return "exact"
    if case["net"] in ("conv", "block", "decoder"):
        return {"rel": 1e-5} if case["dtype"] == "f32" else {"rel": 1.5e-3, "max": 0.2}
    return {"rel": 1e-4, "max": 0.3} if case["dtype"] == "f32" else {"rel": 6e-3, "max": 0.4}


# ---- the same frames in 64 bits, in plain torch --------------------------------------------------------------------------
def _conv64(x, w, nd, bias):
    k, s, p = nd["k"], nd["stride"], nd["pad"]
    n, h, wd, c = x.shape
    oh, ow = (h + 2 * p - k) // s + 1, (wd + 2 * p - k) // s + 1
    x = F.pad(x, (0, 0, p, p, p, p))
    y = torch.zeros((n, oh, ow, nd["cout"]), dtype=torch.float64, device=x.device)
    for dy in range(k):
        for dx in range(k):
            tap = x[:, dy:dy + s * (oh - 1) + 1:s, dx:dx + s * (ow - 1) + 1:s]
            y += tap * w[dy, dx] if nd["depthwise"] else (tap.reshape(-1, c) @ w[dy, dx]).view(y.shape)
    return y if bias is None else y + bias


def _pool64(x, nd):
    return F.max_pool2d(x.permute(0, 3, 1, 2), nd["k"], nd["stride"], nd["pad"]).permute(0, 2, 3, 1)


def _up64(x, nd):
    mode = {"mode": "nearest"} if nd["kind"] == "upsample" else {"mode": "bilinear", "align_corners": False}
    return F.interpolate(x.permute(0, 3, 1, 2), scale_factor=nd["factor"], **mode).permute(0, 2, 3, 1)


def exact(case, seed):
    if case["net"] == "mask_compact":
        return None
    nodes = nodes_of(case)
    weights = {i: [torch.from_numpy(v).cuda().double() for v in wb] for i, wb in _weights(case, nodes, seed).items()}
    clip = _clip(case, seed)
    frames = [clip[1]] if case["first"] else [clip[0], clip[1]]
    kept, O = {}, None
    last_use = {j: i for i, nd in enumerate(nodes) for j in nd["in"]}
    for t, frame in enumerate(frames):
        x, got = frame.double(), {}
        for i, nd in enumerate(nodes):
            kind, dense = nd["kind"], t == 0
            ins = [got[j] for j in nd["in"]]
            f = (lambda v: v.clamp(0, 6)) if nd.get("f") == "relu6" else (lambda v: v.clamp(min=0))
            if kind == "deltagen":
                d = x - kept[i][0] if not dense else x
                new = d.abs().amax(-1, keepdim=True) >= nd["eps"] if not dense else None
                y = d if dense else torch.where(new, d, 0.0)
                kept[i] = [x if dense else torch.where(new, x, kept[i][0])]
            elif kind == "conv":
                y = _conv64(ins[0], weights[i][0], nd, weights[i][1] if dense else None)
            elif kind == "act" and dense:
                kept[i], y = [ins[0], torch.zeros_like(ins[0])], f(ins[0])
            elif kind == "act":
                xa, xt = kept[i]
                s = xa + xt + ins[0]
                y = f(s) - f(xa)
                # (a pixel that nothing reached has s = x^A + x^T, whose change is below the threshold already)
                new = y.abs().amax(-1, keepdim=True) >= nd["eps"]
                kept[i] = [torch.where(new, s, xa), torch.where(new, 0.0, s - xa)]
                y = torch.where(new, y, 0.0)
            elif kind == "add":
                y = ins[0] + ins[1]
            elif kind == "concat":
                y = torch.cat(ins, -1)
            elif kind == "maxpool":
                total = ins[0] if dense else kept[i][0] + ins[0]
                y = _pool64(total, nd) - (0.0 if dense else _pool64(kept[i][0], nd))
                kept[i] = [total]
            elif kind == "accum":
                O = ins[0] if dense else O + ins[0]
                y = O
            else:
                y = _up64(ins[0], nd)
            got[i] = y
            for j in nd["in"]:
                if last_use[j] == i:
                    got.pop(j, None)
    out = {"out": O}
    if case["net"] in ("conv", "block", "decoder"):
        out.update({"state%d" % i: kept[i][0] for i, nd in enumerate(nodes) if nd["kind"] in ("deltagen", "act")})
    return out
