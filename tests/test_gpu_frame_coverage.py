"""Every unit of every frame exactly once, seen in the frames' values: frames in
a row, more than three times around the counters' 64 slots, from two fragment
buffers of different colours in turn, on the routes of the frame's launches
(a workgroup for every unit, tickets, few blocks over few counters, runs of
groups of deep tiles, the entry point without allocation).

Plain frames: the first two against the oracle, every later one the bits of
its buffer's first.  Accumulating frames: mean and M2 against the closed form of
n values a, b, a, b, ... per pixel.  Rounding: a step of the mean rounds within u
|mu| and 2 u |a - b| / k, which the later steps only shrink, so with m = max(|a|,
|b|) the mean is within r = (n + 2 H_n) u m; M2 adds per step at most 2 |a - b| r
+ 2 u (a - b)^2 + u M2, within 2 n r |a - b| + (2 n + n^2 / 4) u (a - b)^2.  A frame
left out or folded in twice moves the mean by |a - b| / 2 n and M2 by (a - b)^2 / 4,
fifty times as far."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_helpers import U32, assert_colour, stream_handle, torch_dev, upload

pytestmark = pytest.mark.gpu

BG = (0.0, 0.0, 0.0, 0.0)  # a background would not alternate
N = 131                    # odd: one more of a than of b


def check_moments(mu, m2, a, b, n):
    """mu [T][P][4], m2 [T][P][3], a and b [T][P][4], float64: the largest error over its bound."""
    na, nb = (n + 1) // 2, n // 2
    mean = (na * a + nb * b) / n
    m, d = np.maximum(np.abs(a), np.abs(b)), np.abs(a - b)
    r = (n + 2 * np.sum(1.0 / np.arange(1, n + 1))) * U32 * m
    m, d, r3 = m[..., :3], d[..., :3], r[..., :3]
    q = 2 * n * r3 * d + (2 * n + n * n / 4) * U32 * d * d
    e = np.abs(mu - mean) / (r + 1e-30)
    e2 = np.abs(m2 - na * nb / n * d * d) / (q + 1e-30)
    return float(e.max()), float(e2.max())


def run(counts, tile, work, waves, op, dtype=np.float32):
    torch = torch_dev()
    import paper_2305_07083_amd as dfb
    n_tiles = len(counts)
    cols = max(d for d in range(1, 101) if n_tiles % d == 0)
    f = workloads.generation_frame(tile * cols, tile * (n_tiles // cols), tile, np.asarray(counts, dtype=np.int32),
                                   7 + n_tiles, depth_by_generation=False).as_dtype(dtype)
    second = f.frag.copy()
    second[:, 0:3] *= dtype(0.5)
    second[:, 3] *= dtype(0.75)
    frags = [upload(f.frag), upload(second)]
    cfg = dfb.make_config(f.width, f.height, tile, work=work, waves=waves, background=BG, op=op,
                          fmt=dfb.DFB_FMT_RGBAF32, dtype=dfb.DFB_F16 if dtype == np.float16 else dfb.DFB_F32)
    out = torch.empty((2, f.n_tiles, f.P, 4), dtype=torch.float32, device="cuda:0")
    got = torch.empty_like(out[0])
    same = torch.ones((), dtype=torch.bool, device="cuda:0")
    with dfb.Compositor(cfg, stream_handle()) as c:
        def frame(k, **kw):
            c.set_fragments(frags[k % 2], f.frag.shape[0], f.layers, f.expected)
            c.composite(**kw)
        for k in range(200):
            frame(k)
            dfb.dfb_read_tiles(c.h, dfb.DFB_BUF_FINAL, 0, f.n_tiles, out[k] if k < 2 else got, True)
            if k >= 2:
                same &= (got == out[k % 2]).all()
        assert bool(same)
        for k in range(N):
            frame(k, accumulate=True)
        assert c.info().accumulation_id == N
        mu = c.read(dfb.DFB_BUF_ACCUM_F32).astype(np.float64)
        m2 = np.moveaxis(c.read(dfb.DFB_BUF_M2_F32).astype(np.float64), 1, 2)
    host = [o.cpu().numpy() for o in out]
    for x, h in zip((f.frag, second), host):
        ref = oracle.composite(x, f.layers, f.width, f.height, tile, tile, expected=f.expected, background=BG,
                               op={0: "blend", 1: "list", 2: "average"}[op], want_mag=True)
        assert_colour(h.reshape(ref["rgba"].shape), ref["rgba"], ref["mag"], "%d tiles" % n_tiles)
    a, b = (h.astype(np.float64).reshape(mu.shape) for h in host)
    e, e2 = check_moments(mu, m2.reshape(a.shape[:2] + (3,)), a, b, N)
    assert e <= 1 and e2 <= 1, (e, e2)
    off, layer_off, kmax = dfb.layer_tables(f.layers, f.n_tiles, f.P)
    off, layer_off = torch.from_numpy(off).cuda(), torch.from_numpy(layer_off).cuda()
    same.fill_(True)
    for k in range(140):
        got.fill_(-1)
        dfb.dfb_composite_noalloc(cfg, frags[k % 2], off, layer_off, kmax, got, stream=stream_handle())
        same &= (got == out[k % 2]).all()
    assert bool(same)


@pytest.mark.parametrize("n_tiles,tile,work,waves", [
    (1, 16, 16, 1),       # one unit
    (1, 64, 16, 4),       # one block of 16 units
    (17, 32, 16, 2),      # 17 blocks over 16 counters
    (256, 32, 16, 4),     # 1024 workgroups
    (2304, 16, 16, 4),    # about as many units as the chip holds workgroups
    (700, 64, 16, 4),     # 11200 units
    (9000, 16, 16, 1),
])
@pytest.mark.parametrize("op", [0, 1, 2])
def test_shallow_frames(n_tiles, tile, work, waves, op):
    run(1 + np.arange(n_tiles) % 4, tile, work, waves, op)


@pytest.mark.parametrize("dtype", [np.float32, np.float16])
@pytest.mark.parametrize("tile,n_tiles,deepest", [(64, 36, 45), (40, 60, 40), (72, 20, 130)])
def test_frames_with_deep_tiles(tile, n_tiles, deepest, dtype):
    rng = np.random.default_rng(tile)
    run(np.where(rng.random(n_tiles) < 0.8, rng.integers(33, deepest + 1, n_tiles), rng.integers(1, 33, n_tiles)), tile,
        tile, 4, 0, dtype)
