"""What this framework is timed on: frames through the encoder and its heads, the way a user's program drives them.

A program builds an `Engine` once (weights, workspace, streams), keeps it, and then hands it frame after frame:
`encode` writes a frame's features, `run_head` reads them in place.  So `prepare` makes the frames of one seed on the
GPU and takes the engine of the case's configuration, which is built on the first request and kept while cases of
that configuration are being prepared; `run` is one pass of frames through it.  Nothing waits for the device.

Models, image sizes, batches and heads of the listed cases are those of `vpe_inputs.CONFIGS`, of `bench.py` and of the
tests; `draw` spreads over the same models with other grids, batches, heads and engine options.
"""
from __future__ import annotations

import math

import torch
import torch.nn.functional as F

import paper_2508_11584_amd as vpe
import vpe_inputs as vi

HEAD_KIND = {"seg": vi.HEAD_SEG, "depth": vi.HEAD_DEPTH, "det": vi.HEAD_DET, "dpt": vi.HEAD_DPT}

#: width, blocks, MLP hidden units, SwiGLU, register tokens, tapped blocks
MODELS = {
    "vits": (384, 12, 1536, False, 0, (3, 6, 9, 12)),
    "vitb": (768, 12, 3072, False, 0, (3, 6, 9, 12)),
    "vitl": (1024, 24, 4096, False, 4, (6, 12, 18, 24)),
    "vitg": (1536, 40, 4096, True, 4, (10, 20, 30, 40)),
}


def _frames(name, model, h, w, batch=1, dtype="bf16", heads="seg,depth,det", every="", head_ch=256, seg_classes=21,
            frames=1, lanes=1, graphs=False, camera=False):
    """A pass of `frames` frames.  lanes: encoder lanes (the ring has one slot more; one lane: the default ring of two).
    camera: frames arrive as 1080p uint8 and are resized and normalised on the encoder's stream first."""
    c = dict(kind="frames", model=model, h=h, w=w, batch=batch, dtype=dtype, heads=heads, every=every, head_ch=head_ch,
             seg_classes=seg_classes, frames=frames, lanes=lanes, graphs=graphs, camera=camera)
    return dict(c, name=name) if name else c


def _transform(name, batch, src_h, src_w, h, w):
    c = dict(kind="transform", batch=batch, src_h=src_h, src_w=src_w, h=h, w=w)
    return dict(c, name=name) if name else c


def listed():
    return [
        # one camera's 1080p frame made into the model's input: the transform in front of every encode
        _transform("camera_1080p", 1, 1080, 1920, 476, 630),
        # the smallest call: one 224 x 224 frame, segmentation only, an engine as it comes (one lane, eager launches)
        _frames("vits_224_seg", "vits", 224, 224, heads="seg"),
        # the same in fp32, for a user who checks numbers against another implementation
        _frames("vits_224_seg_f32", "vits", 224, 224, dtype="f32", heads="seg"),
        # the headline workload (three heads on one 476 x 630 frame) on an engine as it comes: a robot's control loop
        _frames("vits_476x630", "vits", 476, 630),
        # ... as a stream from the camera: frames overlap (two lanes is what a process with the default number of
        # hardware queues is told to use), graphs, 1080p input
        _frames("vits_476x630_stream", "vits", 476, 630, lanes=2, graphs=True, camera=True),
        # ... in fp32 with all heads
        _frames("vits_476x630_f32", "vits", 476, 630, dtype="f32"),
        # ... with the full DPT depth head at its ViT-S width, the paper's own set of heads
        _frames("vits_476x630_dpt", "vits", 476, 630, heads="seg,dpt,det", head_ch=64, graphs=True),
        # heads at rates 1, 2 and 3 over six frames of a moving view
        _frames("vitb_518_rates", "vitb", 518, 518, heads="depth,seg,det", every="1,2,3", frames=6, lanes=2, graphs=True),
        # a foundation module alone (its maps go to somebody else's heads): three odd-sized views
        _frames("vitb_252x406_b3", "vitb", 252, 406, batch=3, heads=""),
        # one view through a large backbone, waited for
        _frames("vitl_518", "vitl", 518, 518, graphs=True),
        # four camera views per step, throughput
        _frames("vitl_518_b4", "vitl", 518, 518, batch=4, lanes=2, graphs=True),
        # the largest: eight views, the largest backbone
        _frames("vitg_518_b8", "vitg", 518, 518, batch=8, seg_classes=150, lanes=2, graphs=True),
    ]


def draw(rng):
    log = lambda lo, hi: math.exp(rng.uniform(math.log(lo), math.log(hi)))  # noqa: E731
    most = _flops(listed()[-1])
    if rng.random() < 0.1:
        return _transform(None, int(log(1, 9)), int(log(240, 2161)), int(log(320, 3841)), 14 * int(log(12, 61)), 14 * int(log(12, 61)))
    while True:
        model = rng.choice(("vits", "vits", "vits", "vitb", "vitb", "vitl", "vitl", "vitg"))
        dtype = "f32" if model in ("vits", "vitb") and rng.random() < 0.2 else "bf16"
        gh = int(log(12, 65))
        gw = min(64, max(12, int(gh * log(0.5, 2.0))))
        batch = int(log(1, 9))
        sets = ["seg", "seg", "depth", "seg,depth", ""]
        if batch * gh * gw >= 900:                      # (a detection class map has one cell per patch)
            sets += ["seg,depth,det", "seg,depth,det", "seg,depth,det", "seg,dpt,det", "det"]
        heads = rng.choice(sets)
        graphs = rng.random() < 0.6
        case = _frames(None, model, 14 * gh, 14 * gw, batch=batch, dtype=dtype, heads=heads,
                       head_ch=64 if "dpt" in heads else rng.choice((128, 256, 256)), seg_classes=rng.choice((21, 21, 150)),
                       lanes=rng.choice((1, 1, 2)), graphs=graphs, camera=rng.random() < 0.2)
        if _flops(case) * (16.0 if dtype == "f32" else 1.0) <= most:
            return case


# ------------------------------------------------------------------ the work of a pass
def _spec(case):
    dim, depth, hidden, gated, registers, taps = MODELS[case["model"]]
    return vi.ModelSpec("case", dim=dim, depth=depth, heads=dim // 64, mlp_hidden=hidden,
                        mlp_kind=vi.MLP_SWIGLU if gated else vi.MLP_GELU, registers=registers, batch=case["batch"],
                        img_h=case["h"], img_w=case["w"], dtype=case["dtype"], taps=taps,
                        seg_classes=case["seg_classes"], head_ch=case["head_ch"])


def _heads(case):
    return [k for k in case["heads"].split(",") if k]


def _every(case):
    return [int(n) for n in case["every"].split(",")] if case["every"] else [1] * len(_heads(case))


def _head_flops(spec, kind):
    D, ch, P = spec.dim, spec.head_ch, spec.batch * spec.patches
    if kind == "seg":
        return 2.0 * P * D * spec.seg_classes
    if kind == "det":
        return 2.0 * P * (9.0 * D * 2 * ch + ch * (spec.det_classes + 4))
    if kind == "depth":
        return 2.0 * P * (4.0 * D * ch + 85.0 * 9 * ch * ch + 64.0 * ch)
    F, oc = ch, [3 * ch // 4 << i for i in range(4)]                 # dpt
    n = [16.0, 4.0, 1.0, 0.25]                                         # cells of the levels per patch
    f = sum(D * c for c in oc) + oc[0] * oc[0] * 16 + oc[1] * oc[1] * 4 + 0.25 * 9 * oc[3] * oc[3]
    f += sum(9.0 * c * F * m for c, m in zip(oc, n))                   # to F channels
    f += 9.0 * F * F * (2 * n[3] + 4 * (n[2] + n[1] + n[0])) + F * F * sum(n)
    f += 9.0 * F * (F // 2) * 64 + (9.0 * (F // 2) * 32 + 32) * 196    # output convolutions
    return 2.0 * P * f


def _flops(case):
    if case["kind"] == "transform":
        return 3.0 * 10 * case["batch"] * case["h"] * case["w"]
    s = _spec(case)
    N, D = s.tokens, s.dim
    T = s.batch * N
    enc = 2.0 * s.batch * s.patches * 588 * D
    enc += s.depth * (2.0 * T * D * (4 * D + s.fc1_out + s.mlp_hidden) + 4.0 * s.batch * N * N * D)
    total = case["frames"] * enc
    for kind, n in zip(_heads(case), _every(case)):
        total += -(-case["frames"] // n) * _head_flops(s, kind)
    return total


def work(case):
    if case["kind"] == "transform":
        return {"bytes": case["batch"] * 3.0 * (case["src_h"] * case["src_w"] + 4.0 * case["h"] * case["w"]), "flops": _flops(case)}
    s = _spec(case)
    esz = 2.0 if s.dtype == "bf16" else 4.0
    pixels, cells = s.batch * s.img_h * s.img_w, s.batch * s.patches
    frame = 3.0 * pixels * 4 + esz * 4 * s.batch * s.tokens * s.dim    # image in, four feature maps out
    if case["camera"]:
        frame += 3.0 * s.batch * 1080 * 1920
    total = case["frames"] * frame + esz * vi.blob_floats(vi.backbone_layout(s))
    for kind, n in zip(_heads(case), _every(case)):
        out = {"seg": 4.0 * cells * s.seg_classes + pixels, "det": 4.0 * cells * (s.det_classes + 4) + cells}.get(kind, 4.0 * pixels)
        total += -(-case["frames"] // n) * out + esz * vi.blob_floats(vi.head_layout(s, HEAD_KIND[kind]))
    return {"bytes": total, "flops": _flops(case)}


def tolerance(case):
    """About four times what the path differs from itself by when its sums run in another order (other GEMM tiles, no
    split k range, other attention shapes).  bf16 features and head outputs: 0.0017 relative (ViT-S), 0.0023 (ViT-B), 0.0043
    (ViT-L), 0.0035 (ViT-g), the full DPT head 0.012 (it amplifies what comes in by its twenty layers); largest single
    difference 0.015, 0.021, 0.026, 0.063, DPT 0.12; class maps: 0.0053 of the cells (near ties).  fp32: 1.2e-6, 5.7e-6,
    none."""
    if case["kind"] == "transform":
        return {"rel": 2e-6, "max": 2e-5}
    dpt = "dpt" in case["heads"]
    if case["dtype"] == "f32":
        return {"rel": 4e-5 if dpt else 5e-6, "max": 4e-4 if dpt else 5e-5, "differ": 0.001}
    rel, most = {"vits": (0.007, 0.06), "vitb": (0.01, 0.08), "vitl": (0.017, 0.1), "vitg": (0.014, 0.25)}[case["model"]]
    return {"rel": 0.03, "max": 0.5, "differ": 0.01} if dpt else {"rel": rel, "max": most, "differ": 0.01}


# ------------------------------------------------------------------ what a program has in hand before the call
def _weights(layout, gen, quantize, std_of=lambda name, shape: 0.02):
    """One flat fp32 blob in the documented order: N(0, std^2) truncated at two deviations, LayerNorm gains around 1,
    LayerScale 0.1, a depth head's output bias at 0.5 (a trained head's depths are positive)."""
    sizes = [math.prod(shape) for _, shape in layout]
    x = torch.empty(sum(sizes), device="cuda")
    torch.nn.init.trunc_normal_(x, std=1.0, a=-2.0, b=2.0, generator=gen)
    at = 0
    for (name, shape), n in zip(layout, sizes):
        t, leaf = x[at:at + n], name.split(".")[-1]
        at += n
        if leaf in ("ls1", "ls2"):
            t.fill_(0.1)
        elif leaf in ("out_b", "head3_b"):
            t.fill_(0.5)
        else:
            t.mul_(std_of(name, shape))
            if leaf in ("ln1_g", "ln2_g", "norm_g"):
                t.add_(1.0)
    if quantize:
        x = x.bfloat16().float()
    return x.cpu().numpy()


def _dpt_std(name, shape):
    """He-sized kernels, so that the signal keeps its size through the head's twenty layers."""
    if name.endswith("_b"):
        return 0.1
    return math.sqrt(2.0 / (shape[0] if name.startswith("up") else math.prod(shape[1:])))


def _blobs(case):
    """The weights of the case's configuration: one blob per head, and the backbone's (in fp32, on the host)."""
    s = _spec(case)
    gen = torch.Generator("cuda").manual_seed(1000 + s.dim)
    quantize = s.dtype == "bf16"
    heads = []
    for kind in _heads(case):
        layout = vi.head_layout(s, HEAD_KIND[kind])
        heads.append(_weights(layout, gen, quantize, _dpt_std) if kind == "dpt" else _weights(layout, gen, quantize))
    return heads, _weights(vi.backbone_layout(s), gen, quantize)


_kept = {}


def _engine(case):
    """The engine of the case's configuration: built once, kept until another configuration is asked for."""
    key = repr(sorted((k, v) for k, v in case.items() if k not in ("name", "frames", "camera")))
    if key not in _kept:
        _kept.clear()
        s, kinds = _spec(case), _heads(case)
        blobs, backbone = _blobs(case)
        cfgs = [vpe.HeadCfg(kind=HEAD_KIND[kind], weights=blob, every_n=n, channels=0 if kind == "seg" else s.head_ch,
                            classes={"seg": s.seg_classes, "det": s.det_classes}.get(kind, 0))
                for kind, blob, n in zip(kinds, blobs, _every(case))]
        lanes = case["lanes"]
        engine = vpe.Engine(dim=s.dim, depth=s.depth, heads=s.heads, mlp_hidden=s.mlp_hidden, mlp_kind=s.mlp_kind,
                            registers=s.registers, img_h=s.img_h, img_w=s.img_w, batch=s.batch,
                            dtype=vpe.VPE_BF16 if s.dtype == "bf16" else vpe.VPE_F32, taps=s.taps, ring_slots=lanes + 1,
                            encoder_lanes=lanes, flags=vpe.VPE_FLAG_GRAPHS if case["graphs"] else 0,
                            weights=backbone, head_cfgs=cfgs)
        # the head's results stay in buffers of the engine: views of them are taken once
        views = {"%d_%s%d" % (i, kind, which): engine.head_output(i, which)
                 for i, kind in enumerate(kinds) for which in range(2 if kind in ("seg", "det") else 1)}
        _kept[key] = (engine, views)
    return _kept[key]


def _field(gen, batch, h, w, frames=1):
    """`frames` pictures of `batch` moving views: per channel a sum of eight random waves, shifted by up to four pixels per
    frame, with fresh noise; fp32 [frames][batch][3][h][w], a few units wide."""
    def uniform(lo, hi):
        return lo + (hi - lo) * torch.rand((1, batch, 3, 8, 1, 1), generator=gen, device="cuda")

    shift = torch.randint(0, 5, (2, frames), generator=gen, device="cuda")
    shift[:, 0] = 0
    dy, dx = shift.cumsum(1).float().view(2, frames, 1, 1, 1, 1, 1)
    y = (torch.arange(h, device="cuda").view(h, 1) + dy) / h
    x = (torch.arange(w, device="cuda").view(1, w) + dx) / w
    amp, fx, fy, phase = uniform(0.5, 1.0), uniform(-4.0, 4.0), uniform(-4.0, 4.0), uniform(0.0, 2.0 * math.pi)
    out = torch.randn((frames, batch, 3, h, w), generator=gen, device="cuda") * 0.05
    for k in range(8):
        out += (amp[:, :, :, k] * torch.sin(2.0 * math.pi * (fx[:, :, :, k] * x[:, :, :, 0] + fy[:, :, :, k] * y[:, :, :, 0]) + phase[:, :, :, k]))
    return out


def _camera_frames(gen, batch, h, w, frames=1):
    """The same views as a camera delivers them: uint8 [frames][batch][h][w][3]."""
    x = (128.0 + 48.0 * _field(gen, batch, h, w, frames)).round_().clamp_(0, 255)
    return x.permute(0, 1, 3, 4, 2).to(torch.uint8).contiguous()


def prepare(case, seed):
    gen = torch.Generator("cuda").manual_seed(seed)
    if case["kind"] == "transform":
        return {"case": case, "frames": _camera_frames(gen, case["batch"], case["src_h"], case["src_w"])[0],
                "out": torch.empty((case["batch"], 3, case["h"], case["w"]), device="cuda")}
    engine, views = _engine(case)
    state = {"case": case, "engine": engine, "views": views, "heads": range(len(_heads(case)))}
    if case["camera"]:
        state["frames"] = list(_camera_frames(gen, case["batch"], 1080, 1920, case["frames"]))
        state["images"] = [torch.empty((case["batch"], 3, case["h"], case["w"]), device="cuda") for _ in state["frames"]]
    else:
        x = _field(gen, case["batch"], case["h"], case["w"], case["frames"])
        x = (x - x.mean((3, 4), keepdim=True)) / x.std((3, 4), keepdim=True)
        state["images"] = list(x)
    return state


# ------------------------------------------------------------------ one pass
def run(state):
    case = state["case"]
    if case["kind"] == "transform":
        vpe.preprocess_u8(state["frames"], state["out"], vi.CAMERA_MEAN, vi.CAMERA_STD)
        return state["out"]
    engine = state["engine"]
    for i, image in enumerate(state["images"]):
        if case["camera"]:
            vpe.preprocess_u8(state["frames"][i], image, vi.CAMERA_MEAN, vi.CAMERA_STD, engine.next_encode_stream())
        frame = engine.encode(image)
        for h in state["heads"]:
            engine.run_head(h, frame)
    return {"features": [engine.feat_view(frame, k) for k in range(4)], **state["views"]}


# ------------------------------------------------------------------ the same in 64 bits, in plain torch
def _named(layout, blob):
    x, at, out = torch.from_numpy(blob).cuda().double(), 0, {}
    for name, shape in layout:
        n = math.prod(shape)
        out[name] = x[at:at + n].view(shape)
        at += n
    return out


def _resized(x, size, aligned=False):
    return F.interpolate(x.permute(0, 3, 1, 2), size=size, mode="bilinear", align_corners=aligned).permute(0, 2, 3, 1)


def _conv3(x, w, b=None, stride=1):
    """3x3, padding 1, of channels-last maps: the nine taps as matrix products."""
    p = F.pad(x, (0, 0, 1, 1, 1, 1))
    H, W = x.shape[1], x.shape[2]
    y = sum(p[:, dy:dy + H:stride, dx:dx + W:stride] @ w[:, :, dy, dx].T.contiguous() for dy in range(3) for dx in range(3))
    return y if b is None else y + b


def _encoded(s, w, image):
    """The four feature maps of one image [3][H][W]."""
    D, heads, eps = s.dim, s.heads, s.ln_eps
    cells = F.unfold(image[None], 14, stride=14)[0].T                   # [P][3 * 14 * 14]
    x = torch.cat((w["cls"][None] + w["pos"][:1], w["reg"], cells @ w["patch_w"].view(D, -1).T + w["patch_b"] + w["pos"][1:]))
    maps = []
    for l in range(s.depth):
        p = {k: w["blk%d.%s" % (l, k)] for k in ("ln1_g", "ln1_b", "qkv_w", "qkv_b", "proj_w", "proj_b", "ls1", "ln2_g",
                                                 "ln2_b", "fc1_w", "fc1_b", "fc2_w", "fc2_b", "ls2")}
        u = F.layer_norm(x, (D,), p["ln1_g"], p["ln1_b"], eps) @ p["qkv_w"] + p["qkv_b"]
        q, k, v = (t.contiguous() for t in u.view(-1, 3, heads, 64).permute(1, 2, 0, 3))
        a = torch.cat([torch.softmax(q[h] @ k[h].T * 0.125, -1) @ v[h] for h in range(heads)], 1)
        x = x + p["ls1"] * (a @ p["proj_w"] + p["proj_b"])
        u = F.layer_norm(x, (D,), p["ln2_g"], p["ln2_b"], eps) @ p["fc1_w"] + p["fc1_b"]
        u = F.silu(u[:, :s.mlp_hidden]) * u[:, s.mlp_hidden:] if s.mlp_kind == vi.MLP_SWIGLU else F.gelu(u)
        x = x + p["ls2"] * (u @ p["fc2_w"] + p["fc2_b"])
        if l + 1 in s.taps:
            maps.append(F.layer_norm(x, (D,), w["norm_g"], w["norm_b"], eps))
    return maps


def _head_exact(s, kind, w, maps):
    """A head's first output from the patch grids [B][gh][gw][D] of the four maps."""
    gh, gw, H, W = s.gh, s.gw, s.img_h, s.img_w
    if kind == "seg":
        return maps[3] @ w["seg_w"].T + w["seg_b"]
    if kind == "det":
        towers = [F.relu(_conv3(maps[3], w[t + "_tower_w"], w[t + "_tower_b"])) for t in ("cls", "box")]
        return torch.cat((towers[0] @ w["cls_w"].T + w["cls_b"], towers[1] @ w["box_w"].T + w["box_b"]), -1)
    if kind == "depth":
        y = 0.0
        for k in range(4):
            size = (gh << k, gw << k)
            z = _resized(maps[3 - k] @ w["proj%d_w" % k].T + w["proj%d_b" % k], size) + y
            z = F.relu(_conv3(z, w["fuse%d_w" % k], w["fuse%d_b" % k]))
            y = _resized(z, (2 * size[0], 2 * size[1])) if k < 3 else _resized(z @ w["out_w"].T, (2 * size[0], 2 * size[1]))
        return F.relu(_resized(y + w["out_b"], (H, W)))[..., 0]
    levels = []
    for i in range(4):
        r = maps[i] @ w["proj%d_w" % i].T + w["proj%d_b" % i]
        if i < 2:                                                        # transposed convolution, kernel = stride = k
            k = 4 >> i
            r = torch.einsum("bhwc,coyx->bhywxo", r, w["up%d_w" % i]).reshape(r.shape[0], gh * k, gw * k, -1) + w["up%d_b" % i]
        elif i == 3:
            r = _conv3(r, w["down3_w"], w["down3_b"], 2)
        levels.append(_conv3(r, w["rn%d_w" % i]))
    unit = lambda x, n: x + _conv3(F.relu(_conv3(F.relu(x), w[n + "_c1_w"], w[n + "_c1_b"])), w[n + "_c2_w"], w[n + "_c2_b"])  # noqa: E731
    path = None
    for k in (3, 2, 1, 0):
        y = levels[k] if path is None else path + unit(levels[k], "fuse%d_a" % k)
        y = unit(y, "fuse%d_b" % k)
        size = levels[k - 1].shape[1:3] if k else (2 * y.shape[1], 2 * y.shape[2])
        path = _resized(y, tuple(size), True) @ w["fuse%d_out_w" % k].T + w["fuse%d_out_b" % k]
    u = _resized(_conv3(path, w["head1_w"], w["head1_b"]), (H, W), True)
    u = F.relu(_conv3(u, w["head2_w"], w["head2_b"]))
    return F.relu(u @ w["head3_w"].T + w["head3_b"])[..., 0]


def exact(case, seed):
    """What `run` leaves behind, in 64 bits (class maps have no such value).  A camera's frame is resized and normalised in
    64 bits as well; weights are those of the engine, in bf16 where it holds them so."""
    mean, std = (torch.tensor(v, dtype=torch.float64, device="cuda").view(3, 1, 1) for v in (vi.CAMERA_MEAN, vi.CAMERA_STD))

    def transformed(frames):
        x = F.interpolate(frames.permute(0, 3, 1, 2).double() / 255.0, size=(case["h"], case["w"]), mode="bilinear", align_corners=False)
        return (x - mean) / std

    gen = torch.Generator("cuda").manual_seed(seed)
    if case["kind"] == "transform":
        return transformed(_camera_frames(gen, case["batch"], case["src_h"], case["src_w"])[0])
    s, kinds = _spec(case), _heads(case)
    if case["camera"]:
        images = [transformed(x) for x in _camera_frames(gen, case["batch"], 1080, 1920, case["frames"])]
    else:
        x = _field(gen, case["batch"], case["h"], case["w"], case["frames"])
        images = [i.double() for i in (x - x.mean((3, 4), keepdim=True)) / x.std((3, 4), keepdim=True)]
    blobs, backbone = _blobs(case)
    w = _named(vi.backbone_layout(s), backbone)
    last = len(images) - 1
    frames = {last - last % n for n in _every(case)} | {last}          # the frames that the outputs belong to
    maps = {f: [torch.stack(m) for m in zip(*(_encoded(s, w, image) for image in images[f]))] for f in frames}
    out = {"features": maps[last]}
    for i, (kind, blob, n) in enumerate(zip(kinds, blobs, _every(case))):
        grids = [m[:, 1 + s.registers:].reshape(s.batch, s.gh, s.gw, s.dim) for m in maps[last - last % n]]
        out["%d_%s0" % (i, kind)] = _head_exact(s, kind, _named(vi.head_layout(s, HEAD_KIND[kind]), blob), grids)
        if kind in ("seg", "det"):
            out["%d_%s1" % (i, kind)] = None
    return out
