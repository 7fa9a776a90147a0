"""The work that users of this library have it do, as timed cases: whole pyramids, the conv stack over
planes of several sizes, the per-window baseline, and single steps of the path, each through a public
entry point of the Python binding.

Sizes are those of paper_1404_1869_amd/configs.py and bench.py (227 x 227 crops, 480 x 640 and 768 x 1024
images, 25 scales on 1200 x 1200 planes, batches of 16, 2000 boxes, fp32 / fp16 / bf16) and, in drawn
cases, others of the same ranges.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch
import torch.nn.functional as F

from paper_1404_1869_amd import densenet as D

MEAN = (123.68, 116.78, 103.94)
LAYERS = ((96, 3, 11, 4, 0, 1), (256, 96, 5, 1, 2, 2), (384, 256, 3, 1, 1, 1), (384, 384, 3, 1, 1, 2),
          (256, 384, 3, 1, 1, 2))  # (M, C, R, stride, pad, groups) of conv1..conv5
LRN_ALPHA, LRN_BETA, LRN_K, LRN_N = 1e-4, 0.75, 1.0, 5
ELEM = {"f32": 4, "f16": 2, "bf16": 2}


# ------------------------------------------------------------------------------------------------
# Cases
# ------------------------------------------------------------------------------------------------
def _pyramid(kind, H, W, scales, spo, dtype, longest=0, pad=0, ramp=False, plane=0, images=1, boxes=0,
             pool5=False):
    return {"kind": kind, "H": H, "W": W, "scales": scales, "spo": spo, "longest": longest, "pad": pad,
            "ramp": ramp, "plane": plane, "images": images, "boxes": boxes, "pool5": pool5, "dtype": dtype}


def listed():
    return [
        # The smallest call: one classifier-sized crop at two scales in fp32 with pool5, through the
        # one-line interface (image in, per-scale maps out), everything planned and allocated by the call.
        dict(_pyramid("featpyramid", 227, 227, 2, 2, "f32", pool5=True), name="featpyramid_227_f32"),
        # The conv stack over the 8 per-scale planes of a 480 x 640 image (no stitching: 8 plane sizes),
        # buffers kept from frame to frame: the 16-bit path of a video loop, and its fp32 twin.
        dict(_pyramid("stack", 480, 640, 8, 4, "f16", longest=1024, pad=16), name="stack_vga_f16"),
        dict(_pyramid("stack", 480, 640, 8, 4, "f32", longest=1024, pad=16), name="stack_vga_f32"),
        # The paper's unit: one image, 25 scales stitched onto 1200 x 1200 planes, 2000 proposals read out.
        dict(_pyramid("pyramid", 768, 1024, 25, 10, "f16", pad=16, ramp=True, plane=1200, boxes=2000),
             name="pyramid_xga_f16"),
        # Throughput serving: a batch of 16 such images with 2000 proposals each (the largest case).
        dict(_pyramid("pyramid", 768, 1024, 25, 10, "bf16", pad=16, ramp=True, plane=1200, images=16,
                      boxes=2000), name="pyramid_xga_x16_bf16"),
        # The per-window baseline the dense pyramid is compared with: 2000 proposals cropped, warped to
        # 227 x 227 and each run through the stack to pool5.
        {"kind": "windows", "H": 768, "W": 1024, "n": 2000, "dtype": "bf16", "name": "windows_x2000_bf16"},
        # Input preparation alone: 16 images packed together onto shared planes.
        dict(_pyramid("build_packed", 768, 1024, 25, 10, "bf16", pad=16, ramp=True, plane=1200, images=16),
             name="build_packed_x16_bf16"),
        # Single layers, for callers with their own schedule: conv1 on a batch of 227 x 227 crops (rows
        # of odd length), conv3 in fp32 on odd-sized maps.
        {"kind": "conv", "layer": 1, "n": 64, "h": 227, "w": 227, "dtype": "f16", "name": "conv1_227_x64_f16"},
        {"kind": "conv", "layer": 3, "n": 8, "h": 37, "w": 49, "dtype": "f32", "name": "conv3_37x49_x8_f32"},
        # Pooling before normalisation (the order of the Caffe reference network) after conv1.
        {"kind": "lrn_pool", "n": 64, "h": 55, "w": 55, "c": 96, "first": False, "dtype": "f16",
         "name": "pool_norm1_x64_f16"},
        # Normalisation before pooling (the default order) after conv2, in fp32.
        {"kind": "lrn_pool", "n": 16, "h": 59, "w": 79, "c": 256, "first": True, "dtype": "f32",
         "name": "norm_pool2_x16_f32"},
        # Proposals of one image read out as max-pooled bins of its conv5 maps.
        dict(_pyramid("region_pool", 768, 1024, 25, 10, "f16", pad=16, ramp=True, plane=1200, boxes=2000),
             name="region_pool_x2000_f16"),
    ]


def _between(rng, lo, hi):
    """A whole number of lo..hi, spread over the logarithm where the range spans more than ten times."""
    if hi > 10 * lo:
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return rng.randint(lo, hi)


def draw(rng):
    kind = rng.choice(("featpyramid", "stack", "pyramid", "windows", "build_packed", "conv", "lrn_pool",
                       "region_pool"))
    half = rng.choice(("f16", "bf16"))
    if kind == "featpyramid":
        return _pyramid(kind, rng.randint(195, 420), rng.randint(195, 420), rng.randint(1, 3), 2,
                        rng.choice(("f32", half)), pad=rng.choice((0, 16)), pool5=rng.random() < 0.5)
    if kind == "stack":
        dtype = rng.choice(("f32", half))
        return _pyramid(kind, rng.randint(240, 720), rng.randint(240, 960), rng.randint(3, 8),
                        rng.choice((3, 4, 5)), dtype, longest=rng.randint(512, 1024), pad=16,
                        ramp=rng.random() < 0.5, pool5=rng.random() < 0.3)
    if kind in ("pyramid", "build_packed", "region_pool"):
        images = 1 if kind == "region_pool" else _between(rng, 1, 12)
        return _pyramid(kind, rng.randint(360, 900), rng.randint(480, 1100), rng.randint(8, 25),
                        rng.choice((5, 10)), half, pad=16, ramp=True, plane=rng.choice((1200, 1200, 1328)),
                        images=images, boxes=0 if kind == "build_packed" else _between(rng, 50, 2000))
    if kind == "windows":
        return {"kind": kind, "H": rng.randint(360, 900), "W": rng.randint(480, 1200),
                "n": _between(rng, 20, 1500), "dtype": half}
    if kind == "conv":
        layer = rng.randint(1, 5)
        side = (67, 600) if layer == 1 else (13, 110) if layer == 2 else (6, 75)
        return {"kind": kind, "layer": layer, "n": _between(rng, 1, 64), "h": rng.randint(*side),
                "w": rng.randint(*side), "dtype": rng.choice(("f32", half, half))}
    c = rng.choice((96, 256))
    return {"kind": "lrn_pool", "n": _between(rng, 1, 64), "h": rng.randint(13, 150), "w": rng.randint(13, 150),
            "c": c, "first": rng.random() < 0.5, "dtype": rng.choice(("f32", half))}


# ------------------------------------------------------------------------------------------------
# Inputs, made from the seed alone
# ------------------------------------------------------------------------------------------------
_TORCH = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _images(gen, n, H, W):
    """uint8 images with the falling spectrum of natural ones: noise at octave-spaced resolutions, the
    coarser ones stronger, with the channels mostly correlated."""
    x = torch.zeros((n, 3, H, W), device="cuda")
    for o in range(7):
        h, w = max(2, H >> o), max(2, W >> o)
        g = torch.randn((n, 1, h, w), generator=gen, device="cuda") + \
            0.4 * torch.randn((n, 3, h, w), generator=gen, device="cuda")
        x += 1.5 ** o * F.interpolate(g, size=(H, W), mode="bilinear", align_corners=False)
    x = x / x.std() * 58.0 + 118.0
    return x.round().clamp(0, 255).to(torch.uint8)


def _weights(gen):
    """conv1..conv5 with the spread that keeps activations level through ReLU, and small biases."""
    out = []
    for M, C, R, _, _, G in LAYERS:
        fan = C // G * R * R
        w = torch.randn((M, C // G, R, R), generator=gen, device="cuda") * math.sqrt(2.0 / fan)
        out.append((w, 0.1 * torch.randn(M, generator=gen, device="cuda") + 0.1))
    return out


def _activations(gen, shape, dtype, scale=20.0):
    """Post-ReLU maps: about a third zeros, the rest half-normal, channels of different strength."""
    g = 0.5 + torch.rand(shape[-1], generator=gen, device="cuda")
    x = torch.randn(shape, generator=gen, device="cuda").add_(0.4).clamp_(min=0).mul_(scale * g)
    return x.to(_TORCH[dtype])


def _boxes(gen, n, H, W):
    """Proposals as the region benchmark has them: log-uniform sizes 32..512 px and aspects 1:3..3:1."""
    u = torch.rand((4, n), generator=gen, device="cuda", dtype=torch.float64)
    size = torch.exp(math.log(32.0) + u[0] * math.log(16.0))
    ar = torch.exp((2 * u[1] - 1) * math.log(3.0))
    bw, bh = (size * ar.sqrt()).clamp(max=W), (size / ar.sqrt()).clamp(max=H)
    x1, y1 = u[2] * (W - bw), u[3] * (H - bh)
    return torch.stack([x1, y1, x1 + bw, y1 + bh], 1).float().contiguous()


def _params(c):
    return D.pyramid_params(c["scales"], c["spo"], base_longest_side=c["longest"], pad=c["pad"],
                            pad_mode=D.DN_PAD_RAMP if c["ramp"] else D.DN_PAD_ZERO, plane_h=c["plane"],
                            plane_w=c["plane"], mean=MEAN)


def _inputs(case, seed):
    """The case's inputs on the GPU: what a caller has before any of this library runs."""
    gen, kind = _gen(seed), case["kind"]
    if kind == "conv":
        C = LAYERS[case["layer"] - 1][1]
        if case["layer"] == 1:
            img = _images(gen, case["n"], case["h"], case["w"]).float()
            x = (img - torch.tensor(MEAN, device="cuda").view(3, 1, 1)).to(_TORCH[case["dtype"]])
        else:
            x = _activations(gen, (case["n"], case["h"], case["w"], C), case["dtype"])
        return {"x": x, "weights": _weights(gen)}
    if kind == "lrn_pool":
        return {"x": _activations(gen, (case["n"], case["h"], case["w"], case["c"]), case["dtype"], 60.0)}
    if kind == "windows":
        return {"images": _images(gen, 1, case["H"], case["W"]), "weights": _weights(gen),
                "boxes": _boxes(gen, case["n"], case["H"], case["W"])}
    n = case["images"]
    out = {"images": _images(gen, n, case["H"], case["W"])}
    if kind not in ("build_packed", "region_pool"):
        out["weights"] = _weights(gen)
    if kind == "region_pool":
        planes, _ = _geometry(case)
        s = _sides(case["plane"])[6]
        out["maps"] = _activations(gen, (len(planes), s, s, 256), case["dtype"], 1.0)
    if case["boxes"]:
        out["boxes"] = torch.cat([_boxes(gen, case["boxes"], case["H"], case["W"]) for _ in range(n)])
        out["box_img"] = torch.arange(n, device="cuda", dtype=torch.int32).repeat_interleave(case["boxes"])
    return out


def prepare(case, seed):
    st = _inputs(case, seed)
    kind, dt = case["kind"], D.DTYPES[case["dtype"]]
    st["case"], st["dt"] = case, dt
    if "weights" in st:
        st["packed"] = D.densenet_pack_weights(st["weights"], dt)
    if kind == "windows":
        st["pw"] = D.PerWindow(case["n"], dt)
    elif kind == "lrn_pool":
        st["net"] = D.net_params(LRN_ALPHA, LRN_BETA, LRN_K, LRN_N, lrn_before_pool=case["first"])
    elif kind == "build_packed":
        st["plan"] = D.BatchPlan(case["images"], case["H"], case["W"], _params(case))
        st["out"] = D.densenet_build_batch(st["images"], st["plan"], dt)
    elif kind == "featpyramid":
        st["p"], st["net"] = _params(case), D.net_params(pool5=case["pool5"])
    elif kind in ("stack", "pyramid"):
        st["p"] = _params(case)
        st["planes"], st["plan"] = D.densenet_build_pyramid(st["images"], st["p"], dt)
        st["cf"] = D.ConvFeatures(st["plan"].image_descs(case["images"]), dt, D.net_params(pool5=case["pool5"]))
    elif kind == "region_pool":
        st["plan"] = D.densenet_plan_pyramid(case["H"], case["W"], _params(case))
        st["descs"] = []
        for j in range(len(st["maps"])):
            d = D.dn_plane_desc()
            d.h, d.w, d.offset = st["maps"].shape[1], st["maps"].shape[2], j * st["maps"][0].numel()
            st["descs"].append(d)
    if kind in ("pyramid", "region_pool"):
        n = len(st["boxes"])
        st["desc"] = torch.empty((n, 256 * 36), dtype=torch.float32, device="cuda")
        st["scale"] = torch.empty(n, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    return st


def run(st):
    case, dt, kind = st["case"], st["dt"], st["case"]["kind"]
    if kind == "conv":
        return D.densenet_conv_layer(case["layer"], st["x"], case["n"], case["h"], case["w"], dt, st["packed"])
    if kind == "lrn_pool":
        return D.densenet_lrn_pool(st["x"], dt, st["net"])
    if kind == "windows":
        return st["pw"](st["images"], st["boxes"], st["packed"], MEAN)
    if kind == "build_packed":
        plan = st["plan"]
        out = D.densenet_build_batch(st["images"], plan, dt, out=st["out"])
        return out[:plan.total_elems]  # the planes (the builder's scratch follows them)
    if kind == "featpyramid":
        pyra = D.convnet_featpyramid(st["images"], st["p"], st["packed"], dt, st["net"])
        return {"conv5": pyra.conv.conv5, "pool5": pyra.conv.pool5} if case["pool5"] else {"conv5": pyra.conv.conv5}
    if kind == "region_pool":
        desc, scale, _ = D.densenet_region_pool(st["maps"], st["descs"], dt, st["plan"], case["pad"],
                                                len(st["descs"]), st["boxes"], box_img=st["box_img"],
                                                out=st["desc"], scale=st["scale"])
        return {"desc": desc, "scale": scale}
    if kind == "stack":  # the planes are in hand; buffers are kept from frame to frame
        conv5, pool5 = st["cf"](st["planes"], st["packed"])
        return {"conv5": conv5, "pool5": pool5} if case["pool5"] else {"conv5": conv5}
    planes, plan = D.densenet_build_pyramid(st["images"], st["p"], dt, out=st["planes"])
    conv5, _ = st["cf"](planes, st["packed"])
    desc, scale, _ = D.densenet_region_windows(conv5, list(st["cf"].c5d), dt, plan, case["pad"],
                                               len(plan.planes), st["boxes"], box_img=st["box_img"],
                                               out=st["desc"], scale=st["scale"])
    return {"conv5": conv5, "desc": desc, "scale": scale}


# ------------------------------------------------------------------------------------------------
# Geometry: scales, stitching and conv5 windows as the header defines them
# ------------------------------------------------------------------------------------------------
def _sides(v):
    """Sides after conv1, pool1, conv2, pool2, conv3, conv4, conv5, pool5."""
    c1 = (v - 11) // 4 + 1
    p1 = (c1 - 2) // 2 + 1
    p2 = (p1 - 2) // 2 + 1
    return c1, p1, p1, p2, p2, p2, p2, (p2 - 2) // 2 + 1


def _up16(v):
    return -(-v // 16) * 16


def _geometry(case, packed=False):
    key = tuple(case[k] for k in ("H", "W", "scales", "spo", "longest", "pad", "plane", "images"))
    return _geometry_of(*key, packed)


@functools.lru_cache(maxsize=64)
def _geometry_of(H, W, scales, spo, longest, pad, plane, images, packed):
    """(planes [(h, w)], entries [dict]) of one image, or of the whole batch when packed."""
    base = longest / max(H, W) if longest else 1.0
    one = []
    for k in range(scales):
        s = base * 2.0 ** (-k / spo)
        h, w = max(1, int(math.floor(H * s + 0.5))), max(1, int(math.floor(W * s + 0.5)))
        one.append({"k": k, "h": h, "w": w, "sy": h / H, "sx": w / W, "rh": h + 2 * pad, "rw": w + 2 * pad})
    if not plane:
        for k, e in enumerate(one):
            e.update(plane=k, y=0, x=0, image=0)
        planes, items = [(e["rh"], e["rw"]) for e in one], one
    else:
        items = [dict(e, image=b, rh=_up16(e["rh"]), rw=_up16(e["rw"]))
                 for b in range(images if packed else 1) for e in one]
        placed = []  # per plane: rectangles (y0, x0, y1, x1) and the free area
        for i in sorted(range(len(items)), key=lambda i: (-items[i]["rh"], -items[i]["rw"], i)):
            e = items[i]
            for j in range(len(placed) + 1):
                if j == len(placed):
                    placed.append([np.zeros((0, 4), np.int64), plane * plane])
                rects, free = placed[j]
                if free < e["rh"] * e["rw"]:
                    continue
                ys, xs = np.unique(np.append(rects[:, 2], 0)), np.unique(np.append(rects[:, 3], 0))
                y, x = (v.ravel() for v in np.meshgrid(ys, xs, indexing="ij"))
                ok = (y + e["rh"] <= plane // 16 * 16) & (x + e["rw"] <= plane // 16 * 16)
                for r in rects:
                    ok &= (y + e["rh"] <= r[0]) | (y >= r[2]) | (x + e["rw"] <= r[1]) | (x >= r[3])
                if ok.any():
                    f = int(np.argmax(ok))
                    e.update(plane=j, y=int(y[f]), x=int(x[f]))
                    placed[j] = [np.vstack([rects, [e["y"], e["x"], e["y"] + e["rh"], e["x"] + e["rw"]]]),
                                 free - e["rh"] * e["rw"]]
                    break
        planes = [(plane, plane)] * len(placed)
    for e in items:  # cells whose centre 16 i + 17.5 lies on a real pixel
        for lo, n, first, last, side in (("y", "h", "r0", "r1", 0), ("x", "w", "c0", "c1", 1)):
            a = e[lo] + pad
            e[first] = max(0, -(-(2 * a - 35) // 32))
            e[last] = min(_sides(planes[e["plane"]][side])[6] - 1, (2 * (a + e[n]) - 36) // 32)
    return planes, items


# ------------------------------------------------------------------------------------------------
# The least work of a pass
# ------------------------------------------------------------------------------------------------
def _conv_flops(h, w, layers=range(5)):
    a, b = _sides(h), _sides(w)
    return sum(2 * M * (C // G) * R * R * a[i] * b[i]
               for (M, C, R, _, _, G), i, l in zip(LAYERS, (0, 2, 4, 5, 6), range(5)) if l in layers)


def work(case):
    kind, es = case["kind"], ELEM[case["dtype"]]
    wbytes = [M * (C // G) * R * R * es for M, C, R, _, _, G in LAYERS]
    if kind == "conv":
        M, C, R, s, p, G = LAYERS[case["layer"] - 1]
        n, h, w = case["n"], case["h"], case["w"]
        ho, wo = ((h - 11) // 4 + 1, (w - 11) // 4 + 1) if case["layer"] == 1 else (h, w)
        return {"bytes": n * (C * h * w + M * ho * wo) * es + wbytes[case["layer"] - 1],
                "flops": 2 * n * M * (C // G) * R * R * ho * wo}
    if kind == "lrn_pool":
        h, w = case["h"], case["w"]
        out = ((h - 2) // 2 + 1) * ((w - 2) // 2 + 1)
        norm = h * w if case["first"] else out
        return {"bytes": case["n"] * case["c"] * (h * w + out) * es,
                "flops": case["n"] * case["c"] * (10 * norm + 8 * out)}
    if kind == "windows":
        n = case["n"]
        return {"bytes": 3 * case["H"] * case["W"] + 16 * n + sum(wbytes) + n * 6 * 6 * 256 * es,
                "flops": n * _conv_flops(227, 227)}
    n = case["images"]
    packed = kind == "build_packed"
    planes, _ = _geometry(case, packed)
    px = sum(h * w for h, w in planes) * (1 if packed else n)
    image = 3 * n * case["H"] * case["W"]
    if packed:
        return {"bytes": image + 3 * px * es, "flops": 3 * px * 8}
    cells = sum(_sides(h)[6] * _sides(w)[6] for h, w in planes) * n
    pool = sum(_sides(h)[7] * _sides(w)[7] for h, w in planes) * n if case["pool5"] else 0
    desc = n * case["boxes"] * (256 * 36 + 1) * 4 + n * case["boxes"] * 20
    if kind == "region_pool":
        return {"bytes": cells * 256 * es + desc, "flops": n * case["boxes"] * 256 * 36 * 6}
    source = 3 * px * es if kind == "stack" else image
    return {"bytes": source + sum(wbytes) + (cells + pool) * 256 * es + desc,
            "flops": n * sum(_conv_flops(h, w) for h, w in planes)}


def tolerance(case):
    """About four times the error against 64 bits that each kind and type was measured to have (the
    rounding of the stored results, and in whole passes of every layer's)."""
    kind, dtype = case["kind"], case["dtype"]
    if kind == "region_pool":
        return "exact"  # maxima of stored values
    if kind == "build_packed":
        return {"rel": {"bf16": 6.5e-3, "f16": 8e-4}[dtype]}
    if kind == "lrn_pool":
        return {"rel": {"bf16": 6.5e-3, "f16": 8.5e-4, "f32": 3e-7}[dtype]}
    if kind == "conv":
        return {"rel": {"bf16": 1e-2, "f16": 1.3e-3, "f32": 3e-6}[dtype]}
    return {"rel": {"bf16": 2.2e-2, "f16": 3e-3, "f32": 4e-6}[dtype], "differ": 1e-4}


# ------------------------------------------------------------------------------------------------
# The same in 64 bits with plain torch
# ------------------------------------------------------------------------------------------------
def _conv64(x, w, b, stride, pad, groups):
    """x [n][C][H][W] -> ReLU(conv), by columns and 2-D products."""
    n, C = x.shape[:2]
    M, Cg, R, _ = w.shape
    ho, wo = (x.shape[2] + 2 * pad - R) // stride + 1, (x.shape[3] + 2 * pad - R) // stride + 1
    out = torch.empty((n, M, ho, wo), dtype=torch.float64, device=x.device)
    step = max(1, (1 << 28) // (Cg * R * R * ho * wo))
    for g in range(groups):
        wg = w[g * M // groups:(g + 1) * M // groups].double().reshape(M // groups, -1)
        for i in range(0, n, step):
            cols = F.unfold(x[i:i + step, g * Cg:(g + 1) * Cg], R, padding=pad, stride=stride)
            m = cols.shape[0]
            cols = cols.permute(1, 0, 2).reshape(Cg * R * R, -1)
            out[i:i + step, g * M // groups:(g + 1) * M // groups] = \
                (wg @ cols).view(M // groups, m, ho, wo).transpose(0, 1)
    return out.add_(b.double().view(1, M, 1, 1)).clamp_(min=0)


def _lrn64(x):
    p = F.pad(x * x, (0, 0, 0, 0, LRN_N // 2, LRN_N // 2))
    s = sum(p[:, j:j + x.shape[1]] for j in range(LRN_N))
    return x * (LRN_K + LRN_ALPHA / LRN_N * s) ** -LRN_BETA


def _pool64(x):
    return F.max_pool2d(x, 3, 2, ceil_mode=True)


def _stack64(x, weights):
    """x [n][3][h][w] fp64 -> conv5 [n][256][Hc][Wc], a few planes at a time."""
    out = []
    step = max(1, int(4e6) // (x.shape[2] * x.shape[3]))
    for i in range(0, x.shape[0], step):
        y = x[i:i + step]
        for l, (w, b) in enumerate(weights):
            y = _conv64(y, w, b, *LAYERS[l][3:])
            if l < 2:
                y = _pool64(_lrn64(y))
        out.append(y)
    return torch.cat(out)


def _taps64(n, size, device):
    """Half-pixel bilinear taps of n outputs over `size` inputs: (first, second, fraction)."""
    o = torch.arange(n, device=device, dtype=torch.float64)
    s = (((2 * o + 1) * size - n) / (2 * n)).clamp(min=0)
    i0 = s.floor()
    return i0.long(), (i0.long() + 1).clamp(max=size - 1), s - i0


def _scale64(img, e, pad, ramp):
    """One padded, centred scale [3][h + 2 pad][w + 2 pad] of an image [3][H][W] fp64."""
    y0, y1, fy = _taps64(e["h"], img.shape[1], img.device)
    x0, x1, fx = _taps64(e["w"], img.shape[2], img.device)
    r = img[:, y0] * (1 - fy)[:, None] + img[:, y1] * fy[:, None]
    v = r[:, :, x0] * (1 - fx) + r[:, :, x1] * fx
    v = v - torch.tensor(MEAN, dtype=torch.float32, device=img.device).double().view(3, 1, 1)
    if not pad:
        return v
    v = F.pad(v[None], (pad,) * 4, mode="replicate")[0]

    def border(n):
        d = torch.arange(-pad, n + pad, device=img.device)
        d = torch.maximum(-d, d - (n - 1)).clamp(min=0).double()
        return ((pad + 1 - d) / (pad + 1)) if ramp else (d == 0).double()
    return v * border(e["h"])[:, None] * border(e["w"])


def _planes64(case, images, packed=False):
    """Planes of every image (or of the packed batch), [3][h][w] fp64 each, image-major."""
    planes, items = _geometry(case, packed)
    out = []
    for b in range(1 if packed else case["images"]):
        mine = [torch.zeros((3, h, w), dtype=torch.float64, device="cuda") for h, w in planes]
        for e in items:
            v = _scale64(images[e["image"] if packed else b].double(), e, case["pad"], case["ramp"])
            mine[e["plane"]][:, e["y"]:e["y"] + v.shape[1], e["x"]:e["x"] + v.shape[2]] = v
        out += mine
    return out


def _choice64(items, boxes):
    """Per box: the entry whose scaled area is closest to 227^2 in ratio (first of equals)."""
    T2 = 227.0 * 227.0
    b = boxes.double()
    bw, bh = b[:, 2] - b[:, 0], b[:, 3] - b[:, 1]
    cost = []
    for e in items:
        area = (e["sy"] * bh) * (e["sx"] * bw)
        c = torch.maximum(area / T2, T2 / area)
        cost.append(c if e["r1"] >= e["r0"] and e["c1"] >= e["c0"] else torch.full_like(c, math.inf))
    return torch.stack(cost).cpu().numpy().argmin(0)


def _span64(items, pick, boxes, pad):
    """Each box on its entry's plane: (top, bottom, left, right) and the entry's fields as tensors."""
    f = {k: torch.tensor([e[k] for e in items], device="cuda")[pick] for k in ("sy", "sx", "y", "x", "r0", "r1",
                                                                                "c0", "c1", "plane")}
    b = boxes.double()
    return (b[:, 1] * f["sy"].double() + f["y"] + pad, b[:, 3] * f["sy"].double() + f["y"] + pad,
            b[:, 0] * f["sx"].double() + f["x"] + pad, b[:, 2] * f["sx"].double() + f["x"] + pad, f)


def _windows64(maps, items, pick, boxes, pad):
    """Bilinear 6 x 6 bin centres of each box: [n][256 * 36]; maps [planes][Hc][Wc][256] fp64."""
    top, bot, left, right, f = _span64(items, pick, boxes, pad)
    q = (torch.arange(6, device="cuda", dtype=torch.float64) + 0.5) / 6

    def cells(lo, hi, first, last):
        g = ((lo[:, None] + q * (hi - lo)[:, None]) - 17.5) * 0.0625
        g = torch.minimum(torch.maximum(g, first[:, None].double()), last[:, None].double())
        i0 = g.floor().long()
        return i0, torch.minimum(i0 + 1, last[:, None]), g - i0
    i0, i1, ly = cells(top, bot, f["r0"], f["r1"])
    j0, j1, lx = cells(left, right, f["c0"], f["c1"])
    p = f["plane"][:, None, None]
    ly, lx = ly[:, :, None, None], lx[:, None, :, None]
    t = maps[p, i0[:, :, None], j0[:, None]] * (1 - lx) + maps[p, i0[:, :, None], j1[:, None]] * lx
    u = maps[p, i1[:, :, None], j0[:, None]] * (1 - lx) + maps[p, i1[:, :, None], j1[:, None]] * lx
    return (t * (1 - ly) + u * ly).permute(0, 3, 1, 2).reshape(len(boxes), -1)


def _bins64(maps, items, pick, boxes, pad):
    """Max-pooled 6 x 6 bins of each box: [n][256 * 36]."""
    top, bot, left, right, f = _span64(items, pick, boxes, pad)

    def ranges(lo, hi, first, last):
        t = torch.arange(6, device="cuda", dtype=torch.float64)
        a = lo[:, None] + (t * (hi - lo)[:, None]) / 6
        z = lo[:, None] + ((t + 1) * (hi - lo)[:, None]) / 6
        i = torch.maximum(((a - 17.5) / 16).ceil().long(), first[:, None])
        j = torch.minimum(((z - 17.5) / 16).ceil().long() - 1, last[:, None])
        near = (((a + z) * 0.5 - 17.5) / 16 + 0.5).floor().long()
        near = torch.minimum(torch.maximum(near, first[:, None]), last[:, None])
        return torch.where(j < i, near, i), torch.where(j < i, near, j)
    i0, i1 = ranges(top, bot, f["r0"], f["r1"])
    j0, j1 = ranges(left, right, f["c0"], f["c1"])
    p = f["plane"][:, None, None]
    out = None
    for di in range(int((i1 - i0).max()) + 1):
        for dj in range(int((j1 - j0).max()) + 1):
            v = maps[p, torch.minimum(i0 + di, i1)[:, :, None], torch.minimum(j0 + dj, j1)[:, None]]
            out = v if out is None else torch.maximum(out, v)
    return out.permute(0, 3, 1, 2).reshape(len(boxes), -1)


def _crops64(image, boxes):
    """Boxes warped to 227 x 227: [n][3][227][227], image [3][H][W] fp64."""
    H, W = image.shape[1:]
    b, o = boxes.double(), torch.arange(227, device="cuda", dtype=torch.float64) + 0.5

    def taps(lo, hi, size):
        s = (lo[:, None] + o * ((hi - lo) / 227)[:, None] - 0.5).clamp(0, size - 1)
        i = s.floor().long()
        return i, (i + 1).clamp(max=size - 1), s - i
    y0, y1, fy = taps(b[:, 1], b[:, 3], H)
    x0, x1, fx = taps(b[:, 0], b[:, 2], W)
    fy, fx = fy[:, :, None], fx[:, None, :]

    def at(y, x):
        return image[:, y[:, :, None], x[:, None, :]].transpose(0, 1)
    fy, fx = fy[:, None], fx[:, None]
    v = (at(y0, x0) * (1 - fx) + at(y0, x1) * fx) * (1 - fy) + (at(y1, x0) * (1 - fx) + at(y1, x1) * fx) * fy
    return v - torch.tensor(MEAN, dtype=torch.float32, device="cuda").double().view(3, 1, 1)


def exact(case, seed):
    st, kind = _inputs(case, seed), case["kind"]
    last = lambda x: x.permute(0, 2, 3, 1).contiguous()  # channels last
    if kind == "conv":
        M, C, R, s, p, G = LAYERS[case["layer"] - 1]
        x = st["x"].double() if case["layer"] == 1 else st["x"].double().permute(0, 3, 1, 2)
        return last(_conv64(x, *st["weights"][case["layer"] - 1], s, p, G))
    if kind == "lrn_pool":
        x = st["x"].double().permute(0, 3, 1, 2)
        return last(_pool64(_lrn64(x)) if case["first"] else _lrn64(_pool64(x)))
    if kind == "windows":
        img = st["images"][0].double()
        parts = [last(_pool64(_stack64(_crops64(img, st["boxes"][i:i + 100]), st["weights"])))
                 for i in range(0, case["n"], 100)]
        return torch.cat(parts)
    if kind == "build_packed":
        pitch = -(-case["plane"] // 64) * 64
        planes = _planes64(case, st["images"], packed=True)
        return torch.cat([F.pad(v, (0, pitch - v.shape[2])).reshape(-1) for v in planes])
    planes, items = _geometry(case)
    if kind == "region_pool":
        pick = _choice64(items, st["boxes"])
        return {"desc": _bins64(st["maps"].double(), items, pick, st["boxes"], case["pad"]),
                "scale": torch.from_numpy(pick.astype(np.int32))}
    source = _planes64(case, st["images"])
    if kind == "stack":  # the planes in hand are already in the storage type
        source = [v.to(_TORCH[case["dtype"]]).double() for v in source]
    if case["plane"]:
        maps = _stack64(torch.stack(source), st["weights"])
        maps = [maps[j:j + 1] for j in range(len(source))]
    else:
        maps = [_stack64(v[None], st["weights"]) for v in source]
    conv5 = torch.cat([last(m).reshape(-1) for m in maps])
    out = {"conv5": conv5}
    if case["pool5"]:
        out["pool5"] = torch.cat([last(_pool64(m)).reshape(-1) for m in maps])
    if case["boxes"]:
        desc, scale = [], []
        n, per = case["boxes"], len(planes)
        for b in range(case["images"]):
            mine = torch.cat([last(m) for m in maps[b * per:(b + 1) * per]])
            boxes = st["boxes"][b * n:(b + 1) * n]
            pick = _choice64(items, boxes)
            desc.append(_windows64(mine, items, pick, boxes, case["pad"]))
            scale.append(pick.astype(np.int32))
        out["desc"], out["scale"] = torch.cat(desc), torch.from_numpy(np.concatenate(scale))
    return out
