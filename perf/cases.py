"""Workloads of the per-tile compositor and its denoiser, for timing and for
comparing results: what a program that owns a framebuffer's tiles has the
library do, over the range of sizes it is used at.

``listed()`` names the cases, ``draw(rng)`` gives another case of the same
ranges, ``prepare(case, seed)`` makes what a program holds before the call,
``run(state)`` is one pass through the public entry points, ``work(case)`` the
bytes and operations a pass cannot do without, and ``exact(case, seed)`` the
same results computed by plain torch in 64 bits.

Kinds of case:
  frame    one composited frame per pass, or with ``frames`` > 0 a progressive
           sequence: the accumulation is reset, that many noisy frames are
           folded in, and the running mean, its M2, the tile variances and the
           display are read out
  noalloc  one frame through the entry point that allocates nothing
  denoise  the U-Net on an accumulated frame
  forward  the U-Net on a batch
  train    one training step of the U-Net and its gradients
"""
import functools
import math

import numpy as np
import torch

import paper_2305_07083_amd as dfb

BACKGROUND = (0.1, 0.2, 0.3, 0.4)
SIGMA = 0.2  # colour noise of a progressive frame


def listed():
    return [
        # The smallest call: four ranks' tiles of a preview-sized frame; what
        # counts is the time from the call to the finished pixels.
        {"name": "preview 256x256, 4 ranks", "kind": "frame", "op": "blend", "content": "uniform", "width": 256,
         "height": 256, "tile": 64, "layers": 4, "dtype": "f32", "format": "rgba8", "frames": 0, "relayout": False},
        # A serving loop that may not allocate: 720p, ragged at both edges.
        {"name": "noalloc 1280x720, 8 ranks", "kind": "noalloc", "op": "blend", "content": "bricks", "width": 1280,
         "height": 720, "tile": 64, "layers": 2, "dtype": "f32", "format": "rgba8", "frames": 0, "relayout": False},
        # An interactive view whose camera moves: every frame brings a new
        # arrival order of its layers, so the layer table is rebuilt.
        {"name": "moving camera 1024x1024", "kind": "frame", "op": "blend", "content": "bricks", "width": 1024,
         "height": 1024, "tile": 64, "layers": 4, "dtype": "f32", "format": "rgba8", "frames": 0, "relayout": True},
        # The benchmark's frame: 64 bricks at 2048x2048, refined progressively
        # while the camera stands still.
        {"name": "progressive 2048x2048", "kind": "frame", "op": "blend", "content": "bricks", "width": 2048,
         "height": 2048, "tile": 64, "layers": 4, "dtype": "f32", "format": "rgba8", "frames": 8, "relayout": False},
        # The wide frame of 256 bricks with planes handed over in half precision.
        {"name": "progressive 4096x1024 f16", "kind": "frame", "op": "blend", "content": "wide bricks", "width": 4096,
         "height": 1024, "tile": 64, "layers": 8, "dtype": "f16", "format": "rgba8", "frames": 4, "relayout": False},
        # Many ranks over one spot, an odd frame size, half precision: layer
        # counts on both sides of the register sort's limit.
        {"name": "deep 1500x1100 f16", "kind": "frame", "op": "blend", "content": "zipf", "width": 1500,
         "height": 1100, "tile": 64, "layers": 128, "dtype": "f16", "format": "rgbaf32", "frames": 0,
         "relayout": False},
        # The largest: 8192x8192 with up to 512 contributors to a tile.
        {"name": "deep 8192x8192", "kind": "frame", "op": "blend", "content": "zipf", "width": 8192, "height": 8192,
         "tile": 128, "layers": 512, "dtype": "f32", "format": "rgbaf32", "frames": 0, "relayout": False},
        # Layers handed over in rank order: blended without a sort.
        {"name": "rank-order list 2048x2048", "kind": "frame", "op": "list", "content": "bricks", "width": 2048,
         "height": 2048, "tile": 64, "layers": 4, "dtype": "f32", "format": "rgba8", "frames": 0, "relayout": False},
        # Redundant renders of some tiles averaged (dynamic load balancing).
        {"name": "average 1920x1080 f16", "kind": "frame", "op": "average", "content": "ragged", "width": 1920,
         "height": 1080, "tile": 64, "layers": 8, "dtype": "f16", "format": "rgba8", "frames": 0, "relayout": False},
        # The benchmark's frame denoised after four accumulated frames.
        {"name": "denoise 2048x2048", "kind": "denoise", "width": 2048, "height": 2048, "n": 4},
        # Inference on a batch of views.
        {"name": "forward 8x256x512", "kind": "forward", "batch": 8, "height": 256, "width": 512},
        # One step of the training loop on its batch of crops.
        {"name": "train 8x128x128", "kind": "train", "batch": 8, "height": 128, "width": 128},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["frame"] * 7 + ["noalloc", "denoise", "forward", "train"])
    if kind == "forward":
        return {"kind": kind, "batch": rng.randint(1, 8), "height": 4 * _log(rng, 4, 128), "width": 4 * _log(rng, 4, 128)}
    if kind == "train":
        return {"kind": kind, "batch": rng.randint(1, 12), "height": 4 * _log(rng, 3, 48), "width": 4 * _log(rng, 3, 48)}
    if kind == "denoise":
        return {"kind": kind, "width": 4 * _log(rng, 16, 512), "height": 4 * _log(rng, 16, 512), "n": rng.randint(1, 5)}
    content = rng.choice(["uniform", "bricks", "bricks", "zipf", "zipf", "ragged"])
    op = "blend"
    if kind == "frame" and content != "bricks":
        op = rng.choice(["blend", "blend", "blend", "list", "average"])
    layers = {"uniform": _log(rng, 1, 40), "bricks": rng.randint(1, 5), "zipf": _log(rng, 8, 400),
              "ragged": _log(rng, 2, 48)}[content]
    frames = rng.choice([0, 0, 0, rng.randint(2, 4)]) if kind == "frame" else 0
    # The sums of a pixel sorted among more than 32 layers are split over
    # lanes by the launch shape, and with them the last bit before a display
    # code is rounded (5 codes of 2.7 million differ between two shapes): such
    # frames are compared in floating point.
    form = rng.choice(["rgba8", "rgbaf32"])
    if op == "blend" and content != "bricks" and layers > 32:
        form = "rgbaf32"
    return {"kind": kind, "op": op, "content": content, "width": _log(rng, 64, 2600), "height": _log(rng, 64, 2600),
            "tile": rng.choice([32, 40, 64, 64, 64, 128]), "layers": layers, "dtype": rng.choice(["f32", "f32", "f16"]),
            "format": form, "frames": frames,
            "relayout": kind == "frame" and frames == 0 and rng.random() < 0.3}


# ------------------------------------------------------------------ layouts
def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _grid(case):
    t = case["tile"]
    return -(-case["width"] // t), -(-case["height"] // t)


@functools.lru_cache(maxsize=4)
def _bricks(width, height, tile, nx, ny, nz):
    """Which tiles each brick of a unit cube's nx x ny x nz decomposition
    projects to under an orthographic camera (azimuth 30, elevation 25), the
    window being the largest rectangle of the frame's aspect inside the cube's
    outline.  Returns tile [L], brick [L], covered [L, P] and depth [L] of the
    brick's centre, ordered by tile, then brick."""
    dev = _device()
    az, el = math.radians(30.0), math.radians(25.0)
    d = -np.array([math.cos(el) * math.cos(az), math.cos(el) * math.sin(az), math.sin(el)])
    u = np.cross(d, [0.0, 0.0, 1.0])
    u /= np.linalg.norm(u)
    v = np.cross(u, d)
    axes = np.stack([u, v], axis=1)  # screen direction of each cube axis
    centre = 0.5 * axes.sum(axis=0)
    half_h = math.inf
    for a in axes:
        n = np.array([-a[1], a[0]]) / np.linalg.norm(a)
        reach = 0.5 * np.abs(axes @ n).sum()
        half_h = min(half_h, reach / (abs(n[0]) * width / height + abs(n[1])))
    half_w = half_h * width / height
    tiles_x, tiles_y = -(-width // tile), -(-height // tile)
    i = torch.arange(tiles_x * tile, device=dev, dtype=torch.float64)
    j = torch.arange(tiles_y * tile, device=dev, dtype=torch.float64)
    X = centre[0] - half_w + (i + 0.5) * (2 * half_w / width)
    Y = centre[1] + half_h - (j + 0.5) * (2 * half_h / height)
    tids, ids, cov, dep = [], [], [], []
    near = [0.0 if c > 0 else 1.0 for c in d]
    for b in range(nx * ny * nz):
        lo = np.array([b % nx / nx, b // nx % ny / ny, b // (nx * ny) / nz])
        hi = lo + np.array([1 / nx, 1 / ny, 1 / nz])
        enter = leave = None
        for k in range(3):
            o = X[None, :] * u[k] + Y[:, None] * v[k]
            t1, t2 = (lo[k] - o) / d[k], (hi[k] - o) / d[k]
            a, z = torch.minimum(t1, t2), torch.maximum(t1, t2)
            enter = a if enter is None else torch.maximum(enter, a)
            leave = z if leave is None else torch.minimum(leave, z)
        hit = (enter < leave).view(tiles_y, tile, tiles_x, tile).permute(0, 2, 1, 3).reshape(tiles_x * tiles_y, -1)
        t = hit.any(dim=1).nonzero()[:, 0]
        tids.append(t)
        ids.append(torch.full_like(t, b))
        cov.append(hit[t])
        dep.append(torch.full((len(t),), float(d @ ((lo + hi) / 2 - near)), device=dev))
    tids, ids, cov, dep = torch.cat(tids), torch.cat(ids), torch.cat(cov), torch.cat(dep)
    order = torch.argsort(tids * (nx * ny * nz) + ids)
    return tids[order].cpu().numpy(), ids[order].cpu().numpy(), cov[order], dep[order].float()


def _counts(case):
    """Layers per tile of the contents without geometry, in descending order
    of the multiset; prepare() deals them to tiles by its seed."""
    tx, ty = _grid(case)
    rng = np.random.default_rng(97)
    if case["content"] == "uniform":
        return np.full(tx * ty, case["layers"])
    if case["content"] == "ragged":  # one tile in ten has none
        return np.where(rng.random(tx * ty) < 0.1, 0, rng.integers(1, case["layers"] + 1, tx * ty))
    # heavy-tailed: truncated Zipf with exponent 1.2, the deepest tile at the cap
    cdf = np.cumsum(np.arange(1, case["layers"] + 1, dtype=np.float64) ** -1.2)
    k = np.searchsorted(cdf / cdf[-1], rng.random(tx * ty), side="right") + 1
    k = np.minimum(k, case["layers"])
    k[0] = case["layers"]
    return k


def _brick_grid(case):
    n = case["layers"]
    return (n, n, n // 2) if case["content"] == "wide bricks" else (n, n, n)


def _layers_in_all(case):
    if "bricks" in case["content"]:
        return len(_bricks(case["width"], case["height"], case["tile"], *_brick_grid(case))[0])
    return int(_counts(case).sum())


def _layout(case, seed):
    """Layer records, tile by tile, source ids ascending; block i is layer i."""
    tx, ty = _grid(case)
    covered = depth = None
    if "bricks" in case["content"]:
        tid, src, covered, depth = _bricks(case["width"], case["height"], case["tile"], *_brick_grid(case))
        counts = np.bincount(tid, minlength=tx * ty)
    else:
        rng = np.random.default_rng([seed, 3])
        counts = rng.permutation(_counts(case))
        tid = np.repeat(np.arange(tx * ty), counts)
        src = np.concatenate([np.sort(rng.permutation(case["layers"])[:k]) for k in counts] or [np.zeros(0)])
    if case["op"] == "list":  # the source id is the generation, from 1
        src = src + 1
    lay = np.empty(len(tid), dtype=dfb.LAYER_DTYPE)
    lay["tile_id"], lay["source_id"], lay["block"] = tid, src, np.arange(len(tid))
    return lay, counts.astype(np.int32), covered, depth


# ------------------------------------------------------------------- inputs
def _generator(seed, what):
    g = torch.Generator(device=_device())
    g.manual_seed(seed * 1000003 + what)
    return g


def _planes(case, seed, covered, depth, n_layers):
    """Fragment planes [L, 5, P]: bricks have alpha ~ Beta(2, 5) where a ray
    hits them and depths that overlap slightly between neighbours; other
    contents alpha, depth ~ U(0, 1).  Colour = alpha * U(0, 1)."""
    dev, P = _device(), case["tile"] ** 2
    dt = torch.float16 if case["dtype"] == "f16" else torch.float32
    out = torch.empty((n_layers, 5, P), dtype=dt, device=dev)
    g = _generator(seed, 1)
    step = max(1, (1 << 26) // P)
    for a in range(0, n_layers, step):
        b = min(n_layers, a + step)
        n = b - a
        if covered is not None:
            two = torch.zeros((n, P), device=dev)
            five = torch.zeros((n, P), device=dev)
            for k in range(7):
                e = torch.empty((n, P), device=dev).exponential_(generator=g)
                (two if k < 2 else five).add_(e)
            alpha = two / (two + five) * covered[a:b]
            z = depth[a:b, None] + 0.01 * torch.rand((n, P), generator=g, device=dev)
        else:
            alpha = torch.rand((n, P), generator=g, device=dev)
            z = torch.rand((n, P), generator=g, device=dev)
        out[a:b, 0:3] = (alpha[:, None] * torch.rand((n, 3, P), generator=g, device=dev)).to(dt)
        out[a:b, 3] = alpha.to(dt)
        out[a:b, 4] = z.to(dt)
    return out


def _noisy(case, seed, base, covered, index):
    """Frame ``index`` of a progressive sequence: colour noise on what is covered."""
    out = base.clone()
    g = _generator(seed, 100 + index)
    step = max(1, (1 << 25) // base.shape[2])
    for a in range(0, base.shape[0], step):
        c = out[a:a + step, 0:3]
        e = torch.randn(c.shape, generator=g, device=base.device) * SIGMA
        if covered is not None:
            e *= covered[a:a + step, None]
        c.copy_((c.float() + e).to(base.dtype))
    return out


def _inputs(case, seed):
    lay, counts, covered, depth = _layout(case, seed)
    base = _planes(case, seed, covered, depth, len(lay))
    if case["frames"]:
        return lay, counts, [_noisy(case, seed, base, covered, i) for i in range(case["frames"])]
    return lay, counts, [base]


def _arrival(lay, seed, which):
    return np.ascontiguousarray(lay[np.random.default_rng([seed, 11, which]).permutation(len(lay))])


def _network_params(seed):
    """He-normal conv weights, small biases and an output layer of a trained
    network's size, flat in the library's order."""
    rng = np.random.default_rng([seed, 5])
    parts = []
    for ci, co in UNET:
        parts.append(rng.standard_normal(9 * ci * co) * math.sqrt(2.0 / (9 * ci)))
        parts.append(rng.standard_normal(co) * 0.05)
    parts += [rng.standard_normal(96) * 0.2, np.zeros(3)]
    return np.concatenate(parts).astype(np.float32)


def _batch(case, seed):
    """Network input [n, h, w, 6] and target: means in (0, 1), log variances
    around -6, a quarter for 1 / n."""
    g, dev = _generator(seed, 2), _device()
    shape = (case["batch"], case["height"], case["width"])
    mean = torch.rand(shape + (4,), generator=g, device=dev)
    logv = torch.randn(shape + (1,), generator=g, device=dev) - 6
    x = torch.cat([mean, logv, torch.full(shape + (1,), 0.25, device=dev)], dim=3).contiguous()
    target = (mean[..., :3] + 0.05 * torch.randn(shape + (3,), generator=g, device=dev)).clamp(0, 1).contiguous()
    return x, target


# ------------------------------------------------------------------ prepare
class _Held:
    """A handle that is closed with the state that holds it."""

    def __init__(self, obj):
        self.obj = obj

    def __del__(self):
        try:
            self.obj.close()
        except Exception:  # the interpreter is going down
            pass


_OPS = {"blend": dfb.DFB_OP_ALPHA_BLEND, "list": dfb.DFB_OP_LIST, "average": dfb.DFB_OP_AVERAGE}
_FORMATS = {"rgba8": dfb.DFB_FMT_RGBA8, "rgbaf32": dfb.DFB_FMT_RGBAF32}
_DTYPES = {"f32": dfb.DFB_F32, "f16": dfb.DFB_F16}


def _config(case, work=0, waves=0):
    return dfb.make_config(case["width"], case["height"], case["tile"], work=work, waves=waves,
                           dtype=_DTYPES[case["dtype"]], fmt=_FORMATS[case["format"]], background=BACKGROUND,
                           op=_OPS[case["op"]])


def _display_like(case, n_tiles, P):
    if case["format"] == "rgba8":
        return torch.empty((n_tiles, P, 4), dtype=torch.uint8, device="cuda")
    return torch.empty((n_tiles, P, 4), dtype=torch.float32, device="cuda")


def _stream():
    return torch.cuda.current_stream().cuda_stream


def _denoise_frames(case):
    return {"kind": "frame", "op": "blend", "content": "bricks", "width": case["width"], "height": case["height"],
            "tile": 64, "layers": 4, "dtype": "f32", "format": "rgba8", "frames": case["n"], "relayout": False}


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind in ("forward", "train"):
        x, target = _batch(case, seed)
        px = case["batch"] * case["height"] * case["width"]
        net = dfb.Denoiser(px, seed=0, stream=_stream())
        dfb.dfb_denoiser_set_params(net.net, _network_params(seed))
        s.update(held=_Held(net), net=net.net, x=x, target=target)
        if kind == "forward":
            s["out"] = torch.empty(x.shape[:3] + (3,), dtype=torch.float32, device="cuda")
        torch.cuda.synchronize()
        return s
    frame = _denoise_frames(case) if kind == "denoise" else case
    lay, counts, frags = _inputs(frame, seed)
    n_tiles, P = len(counts), frame["tile"] ** 2
    s.update(frags=frags, n_blocks=len(lay), counts=counts)
    if kind == "noalloc":
        off, layer_off, kmax = dfb.layer_tables(_arrival(lay, seed, 0), n_tiles, P)
        unit = 32 if frame["tile"] % 32 == 0 else frame["tile"]
        s.update(cfg=_config(frame, work=unit, waves=4), off=torch.from_numpy(off).cuda(),
                 layer_off=torch.from_numpy(layer_off).cuda(), kmax=kmax, display=_display_like(frame, n_tiles, P))
        torch.cuda.synchronize()
        return s
    c = dfb.Compositor(_config(frame), _stream())
    s.update(held=_Held(c), c=c, layers=[_arrival(lay, seed, k) for k in range(2 if frame["relayout"] else 1)],
             display=_display_like(frame, n_tiles, P), turn=0)
    torch.cuda.synchronize()
    # the first frame chooses the launch shape
    for layers in s["layers"]:
        c.set_fragments(frags[0], len(lay), layers, counts)
        c.composite()
    if frame["frames"]:
        for f in frags:
            c.set_fragments(f, len(lay), s["layers"][0], counts)
            c.composite(accumulate=True)
    if kind == "denoise":
        net = dfb.Denoiser(case["width"] * case["height"], seed=0, stream=_stream())
        dfb.dfb_denoiser_set_params(net.net, _network_params(seed))
        s.update(held_net=_Held(net), net=net.net, denoised=torch.empty((n_tiles, P, 4), device="cuda"))
        s["frags"] = None
    elif frame["frames"]:
        s.update(mean=torch.empty((n_tiles, P, 4), device="cuda"), m2=torch.empty((n_tiles, 3, P), device="cuda"),
                 variance=torch.empty(n_tiles, device="cuda"))
    dfb.dfb_synchronize(c.h)
    return s


# ---------------------------------------------------------------------- run
def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "forward":
        dfb.dfb_denoiser_forward(s["net"], s["x"], s["out"], case["batch"], case["height"], case["width"])
        return {"out": s["out"]}
    if kind == "train":
        loss = dfb.dfb_denoiser_train_step(s["net"], s["x"], s["target"], case["batch"], case["height"], case["width"],
                                           1e-4, True)
        return {"loss": np.float32(loss), "gradients": dfb.dfb_denoiser_get_params(s["net"], 1)}
    if kind == "noalloc":
        dfb.dfb_composite_noalloc(s["cfg"], s["frags"][0], s["off"], s["layer_off"], s["kmax"], s["display"],
                                  stream=_stream())
        return {"display": s["display"]}
    c = s["c"]
    n_tiles = c.n_tiles
    if kind == "denoise":
        dfb.dfb_denoise(c.h, s["net"], 1e30)
        dfb.dfb_read_tiles(c.h, dfb.DFB_BUF_DENOISED_F32, 0, n_tiles, s["denoised"], True)
        dfb.dfb_read_tiles(c.h, dfb.DFB_BUF_FINAL, 0, n_tiles, s["display"], True)
        return {"denoised": s["denoised"], "display": s["display"]}
    if case["frames"]:
        c.reset()
        for f in s["frags"]:
            c.set_fragments(f, s["n_blocks"], s["layers"][0], s["counts"])
            c.composite(accumulate=True)
        dfb.dfb_read_tiles(c.h, dfb.DFB_BUF_ACCUM_F32, 0, n_tiles, s["mean"], True)
        dfb.dfb_read_tiles(c.h, dfb.DFB_BUF_M2_F32, 0, n_tiles, s["m2"], True)
        dfb.dfb_read_tiles(c.h, dfb.DFB_BUF_TILE_VARIANCE, 0, n_tiles, s["variance"], True)
        dfb.dfb_read_tiles(c.h, dfb.DFB_BUF_FINAL, 0, n_tiles, s["display"], True)
        return {"mean": s["mean"], "m2": s["m2"], "variance": s["variance"], "display": s["display"]}
    s["turn"] = (s["turn"] + 1) % len(s["layers"])
    c.set_fragments(s["frags"][0], s["n_blocks"], s["layers"][s["turn"]], s["counts"])
    c.composite()
    dfb.dfb_read_tiles(c.h, dfb.DFB_BUF_FINAL, 0, n_tiles, s["display"], True)
    return {"display": s["display"]}


# --------------------------------------------------------------------- work
UNET = [(6, 32), (32, 32), (32, 64), (64, 64), (64, 128), (128, 128), (128, 64), (128, 64), (64, 64), (64, 32),
        (64, 32), (32, 32)]  # (inputs, outputs) of the 3x3 convolutions, in order
UNET_LEVEL = [0, 0, 1, 1, 2, 2, 1, 1, 1, 0, 0, 0]  # halvings of the resolution they run at
UNET_PARAMS = sum(9 * ci * co + co for ci, co in UNET) + 99
UNET_FLOPS = sum(18.0 * ci * co / 4 ** lv for (ci, co), lv in zip(UNET, UNET_LEVEL)) + 192.0  # per pixel, forward


def work(case):
    kind = case["kind"]
    if kind == "denoise":  # reads the mean, writes the denoised pixels and the display
        px = case["width"] * case["height"]
        return {"bytes": px * 36.0 + 4.0 * UNET_PARAMS, "flops": UNET_FLOPS * px}
    if kind in ("forward", "train"):
        px = case["batch"] * case["height"] * case["width"]
        if kind == "forward":
            return {"bytes": px * 36.0 + 4.0 * UNET_PARAMS, "flops": UNET_FLOPS * px}
        # weights, their gradients and both moments are read and written
        return {"bytes": px * 36.0 + 28.0 * UNET_PARAMS, "flops": 3 * UNET_FLOPS * px}
    tx, ty = _grid(case)
    P = case["tile"] ** 2
    px, frags = tx * ty * P, _layers_in_all(case) * P
    planes = 5 if case["op"] == "blend" else 4
    per_frame = frags * planes * (2 if case["dtype"] == "f16" else 4) + px * (4 if case["format"] == "rgba8" else 16)
    n = max(1, case["frames"])
    total = per_frame * n + (case["frames"] and px * (56 * n - 28) + 4 * tx * ty)  # mean and M2 of every frame
    return {"bytes": float(total), "flops": 10.0 * frags * n}


# -------------------------------------------------------------------- exact
def _composite64(case, lay, counts, frag):
    """Every tile composited in 64 bits: [T, P, 4]."""
    dev, P = frag.device, frag.shape[2]
    bg = torch.tensor(BACKGROUND, dtype=torch.float64, device=dev)
    out = bg.expand(len(counts), P, 4).clone()
    first = np.cumsum(counts) - counts  # layers lie tile by tile, source ids ascending
    for k in np.unique(counts):
        tiles = np.nonzero(counts == k)[0]
        step = max(1, (1 << 25) // (int(k) * P or 1))
        for a in range(0, len(tiles) if k else 0, step):
            t = tiles[a:a + step]
            idx = torch.from_numpy(first[t][:, None] + np.arange(k)).to(dev)
            f = frag[idx]  # [n, k, 5, P]
            if case["op"] == "average":
                out[torch.from_numpy(t).to(dev)] = f[:, :, :4].double().mean(dim=1).transpose(1, 2)
                continue
            if case["op"] == "list":
                f = f.flip(1)[:, :, :4].double()
            else:
                # transposed so that a pixel's depths are contiguous for the sort
                order = torch.sort(f[:, :, 4].transpose(1, 2).contiguous(), dim=2, stable=True).indices.transpose(1, 2)
                f = torch.gather(f[:, :, :4], 1, order[:, :, None].expand(-1, -1, 4, -1)).double()
            T = torch.cumprod(1 - f[:, :, 3], dim=1)
            w = torch.cat([torch.ones_like(T[:, :1]), T[:, :-1]], dim=1)
            c = (w[:, :, None] * f).sum(dim=1).transpose(1, 2)
            out[torch.from_numpy(t).to(dev)] = c + T[:, -1, :, None] * bg
    return out


def _accumulate64(case, lay, counts, frags):
    """Running mean, M2 and per-tile variance of the mean of the frames."""
    x = torch.stack([_composite64(case, lay, counts, f) for f in frags])
    mean = x.mean(dim=0)
    m2 = (x[..., :3] - mean[..., :3]).square().sum(dim=0).transpose(1, 2).contiguous()
    n, (tx, ty), t = len(frags), _grid(case), case["tile"]
    inside = torch.zeros((ty * t, tx * t), dtype=torch.float64, device=mean.device)
    inside[:case["height"], :case["width"]] = 1
    inside = inside.view(ty, t, tx, t).permute(0, 2, 1, 3).reshape(tx * ty, t * t)
    if n < 2:
        return mean, m2, torch.full((tx * ty,), math.inf, dtype=torch.float64, device=mean.device)
    var = (m2 * inside[:, None]).sum(dim=(1, 2)) / (3 * inside.sum(dim=1) * n * (n - 1))
    return mean, m2, var


def _conv64(x, w, b):
    n, h, wd, ci = x.shape
    xp = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1))
    y = b
    for r in range(3):
        for c in range(3):
            y = y + xp[:, r:r + h, c:c + wd].reshape(-1, ci) @ w[r, c]
    return torch.relu(y).view(n, h, wd, -1)


def _up64(x):
    return x.repeat_interleave(2, dim=1).repeat_interleave(2, dim=2)


def _pool64(x):
    n, h, w, c = x.shape
    return x.view(n, h // 2, 2, w // 2, 2, c).mean(dim=(2, 4))


def _network64(flat, x):
    p, o = [], 0
    for ci, co in UNET:
        p.append((flat[o:o + 9 * ci * co].view(3, 3, ci, co), flat[o + 9 * ci * co:o + 9 * ci * co + co]))
        o += 9 * ci * co + co
    out_w, out_b = flat[o:o + 96].view(32, 3), flat[o + 96:o + 99]
    s1 = _conv64(_conv64(x, *p[0]), *p[1])
    s2 = _conv64(_conv64(_pool64(s1), *p[2]), *p[3])
    h = _conv64(_conv64(_pool64(s2), *p[4]), *p[5])
    h = torch.cat([_conv64(_up64(h), *p[6]), s2], dim=3)
    h = _conv64(_conv64(h, *p[7]), *p[8])
    h = torch.cat([_conv64(_up64(h), *p[9]), s1], dim=3)
    h = _conv64(_conv64(h, *p[10]), *p[11])
    return x[..., :3] + (h.reshape(-1, 32) @ out_w + out_b).view(x.shape[:3] + (3,))


def exact(case, seed):
    kind = case["kind"]
    if kind in ("forward", "train"):
        x, target = _batch(case, seed)
        flat = torch.from_numpy(_network_params(seed)).to(x.device).double()
        if kind == "forward":
            return {"out": _network64(flat, x.double())}
        flat.requires_grad_(True)
        loss = (_network64(flat, x.double()) - target.double()).square().mean()
        loss.backward()
        return {"loss": loss.detach().cpu().numpy(), "gradients": flat.grad.cpu().numpy()}
    frame = _denoise_frames(case) if kind == "denoise" else case
    lay, counts, frags = _inputs(frame, seed)
    if kind == "denoise":
        mean, _, var = _accumulate64(frame, lay, counts, frags)
        (tx, ty), t, n = _grid(frame), frame["tile"], frame["frames"]
        H, W = case["height"], case["width"]
        image = mean.view(ty, tx, t, t, 4).permute(0, 2, 1, 3, 4).reshape(ty * t, tx * t, 4)
        logv = torch.log(var.clamp_min(1e-12)) if n >= 2 else torch.zeros_like(var)
        logv = logv.view(ty, 1, tx, 1).expand(ty, t, tx, t).reshape(ty * t, tx * t)
        x = torch.cat([image, logv[..., None], torch.full_like(logv[..., None], 1.0 / n)], dim=2)
        flat = torch.from_numpy(_network_params(seed)).to(x.device).double()
        image = image.clone()
        image[:H, :W, :3] = _network64(flat, x[None, :H, :W])[0]
        image = image.view(ty, t, tx, t, 4).permute(0, 2, 1, 3, 4).reshape(tx * ty, t * t, 4)
        return {"denoised": image, "display": None}
    if case["frames"]:
        mean, m2, var = _accumulate64(case, lay, counts, frags)
        return {"mean": mean, "m2": m2, "variance": var, "display": mean if case["format"] == "rgbaf32" else None}
    if case["format"] == "rgba8":
        return None  # codes only
    return {"display": _composite64(case, lay, counts, frags[0])}
