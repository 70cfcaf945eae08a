"""What this library's performance is measured on: the calls that a program
makes through its public entry points, over the sizes, types, borders and
layouts that it serves.

`listed()` names fixed cases, `draw()` gives more of the same ranges; a case
is prepared once (`prepare`) and then run any number of times (`run`).
`work()` counts the bytes and operations one run cannot do without, and
`exact()` is the same operator in 64 bits, in plain torch.
"""
from __future__ import annotations

import math

import numpy as np
import torch
import torch.nn.functional as F

from paper_2305_00515_amd import api
from paper_2305_00515_amd.autograd import sobel4x5_magnitude

DIR_BYTES = {api.DIR_NONE: 0, api.DIR_S16: 2, api.DIR_S32: 4}
PAD_MODE = {api.BORDER_REPLICATE: "replicate", api.BORDER_ZERO: "constant", api.BORDER_REFLECT101: "reflect"}

# The four directional filters, 0, 45, 90 and 135 degrees, and the 3x3 pair.
SOBEL5 = np.array([
    [[-1, -2, 0, 2, 1], [-4, -8, 0, 8, 4], [-6, -12, 0, 12, 6], [-4, -8, 0, 8, 4], [-1, -2, 0, 2, 1]],
    [[-6, -4, -1, -2, 0], [-4, -12, -8, 0, 2], [-1, -8, 0, 8, 1], [-2, 0, 8, 12, 4], [0, 2, 1, 4, 6]],
    [[-1, -4, -6, -4, -1], [-2, -8, -12, -8, -2], [0, 0, 0, 0, 0], [2, 8, 12, 8, 2], [1, 4, 6, 4, 1]],
    [[0, -2, -1, -4, -6], [2, 0, -8, -12, -4], [1, 8, 0, -8, -1], [4, 12, 8, 0, -2], [6, 4, 1, 2, 0]],
])
SOBEL3 = np.array([[[-1, 0, 1], [-2, 0, 2], [-1, 0, 1]], [[-1, -2, -1], [0, 0, 0], [1, 2, 1]]])


def image_case(name, h, w, *, op=api.OP_4DIR_5X5, border=api.BORDER_REPLICATE, dirs=api.DIR_NONE, weights="",
               padded=False):
    return {"name": name, "kind": "image", "h": h, "w": w, "op": op, "border": border, "dirs": dirs,
            "weights": weights, "padded": padded}


def listed():
    return [
        # A thumbnail or a camera crop: the smallest image the operator is compared on; launch latency.
        image_case("mag_512", 512, 512),
        # One video frame, rows back to back.
        image_case("mag_1080p", 1080, 1920),
        # A photograph of odd size, rows back to back (no row aligned), mirrored border.
        image_case("mag_odd_photo", 2999, 4001, border=api.BORDER_REFLECT101),
        # A large scan or a satellite tile: the headline size.
        image_case("mag_8192", 8192, 8192),
        # Orientation features: the magnitude and all four directional responses as int16.
        image_case("planes_s16_4096", 4096, 4096, dirs=api.DIR_S16),
        # The classic 3x3 pair on a 4K frame.
        image_case("op3x3_2160p", 2160, 3840, op=api.OP_2DIR_3X3),
        # Another member of the 5x5 family, weights given at run time, on a 4K frame.
        image_case("weighted_2160p", 2160, 3840, weights="1 3 5 10"),
        # The same with its directional responses, int32, paper-native border.
        image_case("weighted_planes_2048", 2048, 2048, weights="1 3 5 10", dirs=api.DIR_S32,
                   border=api.BORDER_VALID),
        # A plan kept over a fixed set of pictures of many sizes, launched again and again.
        {"name": "plan_48_mixed", "kind": "plan", "count": 48, "lo": 128, "hi": 4096, "sizes": 77,
         "border": api.BORDER_REPLICATE, "dirs": api.DIR_NONE, "padded": True},
        # Detector crops of one frame: a list of small tensors of ragged sizes, one call.
        {"name": "batch_16_crops", "kind": "batch", "count": 16, "lo": 64, "hi": 640, "sizes": 5,
         "border": api.BORDER_REPLICATE, "dirs": api.DIR_NONE, "padded": False},
        # An edge loss in training: fp32 magnitudes and the gradient of the images.
        {"name": "f32_train_32x1024", "kind": "f32", "batch": 32, "h": 1024, "w": 1024,
         "border": api.BORDER_REPLICATE, "grad": True},
        # Decoded frames in host memory through the copy/compute pipeline.
        {"name": "pipe_8x1080p", "kind": "pipe", "count": 8, "h": 1080, "w": 1920,
         "border": api.BORDER_REPLICATE},
    ]


def _side(rng, lo, hi):
    """A side of an image: spread over the logarithm, now and then a multiple of 64, mostly not."""
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return max(lo, v // 64 * 64) if rng.random() < 0.3 else v


def draw(rng):
    kind = rng.choice(["image"] * 6 + ["plan"] * 2 + ["batch"] * 2 + ["f32"] * 3 + ["pipe"])
    border = rng.choice([api.BORDER_REPLICATE, api.BORDER_REPLICATE, api.BORDER_VALID, api.BORDER_ZERO,
                         api.BORDER_REFLECT101])
    padded = rng.random() < 0.3
    if kind == "image":
        form = rng.choice(["mag", "mag", "mag", "planes", "op", "weights"])
        dirs = rng.choice([api.DIR_S16, api.DIR_S32]) if form == "planes" or rng.random() < 0.2 else api.DIR_NONE
        top = 8192 if form == "mag" and dirs == api.DIR_NONE else 4096
        c = {"kind": kind, "h": _side(rng, 64, top), "w": _side(rng, 64, top), "op": api.OP_4DIR_5X5,
             "border": border, "dirs": dirs, "weights": "", "padded": padded}
        if form == "op":
            c["op"] = rng.choice([api.OP_2DIR_5X5, api.OP_2DIR_3X3])
        if form == "weights":   # int16 planes take weights of small sums only
            c["weights"] = "1 2 4 6" if dirs == api.DIR_S16 else rng.choice(["1 3 5 10", "2 3 4 8", "1 2 4 6"])
        return c
    if kind in ("plan", "batch"):
        lo = rng.choice([32, 64, 128])
        dirs = api.DIR_S16 if kind == "plan" and rng.random() < 0.3 else api.DIR_NONE
        most = 32 if kind == "batch" else 12 if dirs else 48
        return {"kind": kind, "count": rng.randint(4, most), "lo": lo,
                "hi": _side(rng, 4 * lo, 3000 if kind == "plan" else 1024), "sizes": rng.randint(0, 9999),
                "border": border, "dirs": dirs, "padded": rng.random() < 0.5}
    if kind == "f32":
        h, w = _side(rng, 48, 2048), _side(rng, 48, 2048)
        return {"kind": kind, "batch": rng.randint(1, max(1, min(32, (8 << 20) // (h * w)))), "h": h, "w": w,
                "border": border, "grad": rng.random() < 0.7}
    return {"kind": kind, "count": rng.randint(2, 8), "h": _side(rng, 240, 1080), "w": _side(rng, 320, 1920),
            "border": border}


# ------------------------------------------------------------------ inputs


def _picture(h, w, gen):
    """A photograph's stand-in as float64 values in [0, 255]: a smooth field,
    filled rectangles with sharp edges, and sensor noise of a few grey levels."""
    dev = gen.device
    grid = torch.rand((1, 1, 9, 9), generator=gen, device=dev) * 160 + 48
    img = F.interpolate(grid, size=(h, w), mode="bilinear", align_corners=True)[0, 0]
    r = torch.rand((12, 5), generator=gen, device=dev).tolist()
    for a, b, c, d, v in r:
        y, x = int(a * h), int(b * w)
        img[y:y + max(4, int(c * h / 3)), x:x + max(4, int(d * w / 3))] += v * 120 - 60
    return (img + 2.0 * torch.randn((h, w), generator=gen, device=dev)).clamp_(0, 255)


def _u8_image(h, w, gen, padded=False):
    img = _picture(h, w, gen).round_().to(torch.uint8)
    if not padded:
        return img
    rows = torch.empty((h, (w + 255) // 256 * 256), dtype=torch.uint8, device=img.device)
    rows[:, :w] = img
    return rows[:, :w]


def _sizes(case):
    r = np.random.default_rng(case["sizes"])
    s = r.integers(case["lo"], case["hi"] + 1, size=(case["count"], 2))
    return [(int(a), int(b)) for a, b in s]


def _weights(text):
    return api.family_weights(*api.family_products(*text.split()))


def _inputs(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    kind = case["kind"]
    if kind == "image":
        return _u8_image(case["h"], case["w"], gen, case["padded"])
    if kind in ("plan", "batch"):
        return [_u8_image(h, w, gen, case["padded"]) for h, w in _sizes(case)]
    if kind == "f32":
        x = torch.stack([_picture(case["h"], case["w"], gen) for _ in range(case["batch"])]) / 255
        ho, wo = api.out_shape(case["h"], case["w"], case["border"])
        return x, torch.randn((case["batch"], ho, wo), generator=gen, device="cuda")
    return [_u8_image(case["h"], case["w"], gen).cpu().numpy() for _ in range(case["count"])]


def prepare(case, seed):
    kind, data = case["kind"], _inputs(case, seed)
    state = {"case": case, "data": data}
    if kind == "image" and case["weights"]:
        state["weights"] = _weights(case["weights"])
    elif kind == "plan":
        shapes = [api.out_shape(*s.shape, case["border"]) for s in data]
        mags = [torch.empty(s, dtype=torch.uint8, device="cuda") for s in shapes]
        dirs = None
        if case["dirs"]:
            dirs = [[torch.empty(s, dtype=torch.int16, device="cuda") for _ in range(4)] for s in shapes]
        state["plan"] = api.Plan(data, mags, case["border"], dir_type=case["dirs"], dirs=dirs)
        state["out"] = [mags, dirs] if case["dirs"] else mags
    elif kind == "f32":
        data[0].requires_grad_(case["grad"])
    elif kind == "pipe":
        state["pipe"] = api.Pipe(case["w"], case["h"])
    return state


def run(state):
    case, data = state["case"], state["data"]
    kind, border = case["kind"], case["border"]
    if kind == "image":
        if case["weights"]:
            return api.sobel4x5_u8_weighted(data, state["weights"], border, dir_type=case["dirs"])
        if case["op"] != api.OP_4DIR_5X5:
            return api.sobel4x5_u8_op(data, case["op"], border, dir_type=case["dirs"])
        return api.sobel4x5_u8(data, border, dir_type=case["dirs"])
    if kind == "plan":
        state["plan"].launch()
        return state["out"]
    if kind == "batch":
        return api.sobel4x5_batched(data, border=border)
    if kind == "f32":
        x, g = data
        m = sobel4x5_magnitude(x, border)
        return (m, torch.autograd.grad(m, x, g)[0]) if case["grad"] else m
    return state["pipe"].run(data, border=border)


# ------------------------------------------------------------- what it takes


def work(case):
    """Bytes: each input read once, each output written once.  Operations: the
    filters in their factored forms (two additions or one multiply-add per
    distinct term), the squares and the root."""
    kind = case["kind"]
    if kind == "f32":
        ho, wo = api.out_shape(case["h"], case["w"], case["border"])
        px, out = case["batch"] * case["h"] * case["w"], case["batch"] * ho * wo
        # forward: x, M; backward: x, dM, dx
        return {"bytes": 4 * (px + out) + (4 * (2 * px + out) if case["grad"] else 0),
                "flops": 35 * px + (80 * px if case["grad"] else 0)}
    op, dirs = case.get("op", api.OP_4DIR_5X5), case.get("dirs", api.DIR_NONE)
    if kind == "pipe":
        sizes = [(case["h"], case["w"])] * case["count"]
    else:
        sizes = _sizes(case) if kind in ("plan", "batch") else [(case["h"], case["w"])]
    planes = 4 if op == api.OP_4DIR_5X5 else 2
    ops = {api.OP_4DIR_5X5: 35, api.OP_2DIR_5X5: 18, api.OP_2DIR_3X3: 12}[op]
    nbytes = flops = 0
    for h, w in sizes:
        ho, wo = api.out_shape(h, w, case["border"], op)
        nbytes += h * w + ho * wo * (1 + planes * DIR_BYTES[dirs])
        flops += ops * ho * wo
    return {"bytes": nbytes, "flops": flops}


def _responses(x, border, filters):
    """Directional responses (B, Ho, Wo), float64, of x (B, H, W)."""
    n = filters.shape[1]
    h, w = api.out_shape(x.shape[1], x.shape[2], border, api.OP_2DIR_3X3 if n == 3 else api.OP_4DIR_5X5)
    if border != api.BORDER_VALID:
        x = F.pad(x[:, None], (n // 2,) * 4, mode=PAD_MODE[border])[:, 0]
    out = []
    for k in filters.tolist():
        g = 0
        for i in range(n):
            for j in range(n):
                if k[i][j]:
                    g = g + k[i][j] * x[:, i:i + h, j:j + w]
        out.append(g)
    return out


def _exact_u8(img, border, filters, dirs):
    g = _responses(img[None].double(), border, filters)
    mag = sum(v * v for v in g).sqrt().round().clamp(max=255).to(torch.uint8)[0]
    return mag, ([v[0].to(torch.int16 if dirs == api.DIR_S16 else torch.int32) for v in g] if dirs else None)


def exact(case, seed):
    kind, border, data = case["kind"], case["border"], _inputs(case, seed)
    if kind == "image":
        filters = SOBEL5
        if case["op"] != api.OP_4DIR_5X5:
            filters = SOBEL3 if case["op"] == api.OP_2DIR_3X3 else SOBEL5[[0, 2]]
        if case["weights"]:
            a, b, n, m = (int(v) for v in case["weights"].split())
            filters = _family(a, b, n, m)
        return _exact_u8(data, border, filters, case["dirs"])
    if kind == "plan":
        got = [_exact_u8(s, border, SOBEL5, case["dirs"]) for s in data]
        mags = [m for m, _ in got]
        return [mags, [d for _, d in got]] if case["dirs"] else mags
    if kind in ("batch", "pipe"):
        return [_exact_u8(torch.as_tensor(s, device="cuda"), border, SOBEL5, api.DIR_NONE)[0] for s in data]
    mags, grads = [], []
    for x, g in zip(*data):      # image by image: the 64-bit graph of a whole batch is large
        x = x[None].double().requires_grad_(case["grad"])
        s = sum(v * v for v in _responses(x, border, SOBEL5))
        m = torch.where(s > 0, s, torch.ones_like(s)).sqrt() * (s > 0)   # no gradient where M = 0
        mags.append(m.detach()[0])
        if case["grad"]:
            grads.append(torch.autograd.grad(m, x, g[None].double())[0][0])
    mag = torch.stack(mags)
    return (mag, torch.stack(grads)) if case["grad"] else mag


def _family(a, b, n, m):
    """The four kernels of the family with whole parameters a, b, n, m."""
    col, side = np.array([1, n, m, n, 1]), np.array([-1, -b, 0, b, 1])
    kx = a * np.outer(col, side)
    kd = a * np.array([[-m, -n, -1, -b, 0], [-n, -m * b, -n * b, 0, b], [-1, -n * b, 0, n * b, 1],
                       [-b, 0, n * b, m * b, n], [0, b, 1, n, m]])
    return np.stack([kx, kd, kx.T, kd[:, ::-1]])
