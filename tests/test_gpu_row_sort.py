"""Tiles of 33 to 512 layers, sorted in registers by 16 lanes a pixel, and the
frames that mix them with the other paths: the edges of every keys-per-lane
class, ragged groups of 32 pixels, tiles and buffers whose planes are not
4-pixel aligned (the LDS sort takes those), accumulation, and layouts that
need the row sort only now and then.  Against the oracle: order bit-exact,
colour within 1e-5 of the magnitude sum, mean, M2 and variance within the
FP32 Welford bound."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_helpers import (WelfordBound, assert_colour, order_as_sources, stream_handle, torch_dev, upload)

pytestmark = pytest.mark.gpu

EDGES = [33, 48, 64, 65, 96, 97, 128, 129, 192, 193, 256, 257, 384, 385, 511, 512, 513]


@pytest.fixture(scope="module")
def dfb():
    torch_dev()
    import paper_2305_07083_amd as m
    m.load()
    return m


def frame_of(counts, tile, seed, dtype=np.float32, ties=False):
    f = workloads.generation_frame(tile * len(counts), tile, tile, counts, seed, depth_by_generation=False)
    if ties:  # a handful of depth values: most comparisons fall to the source id
        f.frag[:, 4] = np.round(f.frag[:, 4] * 16) / 16
    return f.as_dtype(dtype)


def config(dfb, f, **kw):
    dt = dfb.DFB_F16 if f.frag.dtype == np.float16 else dfb.DFB_F32
    return dfb.make_config(f.width, f.height, f.tile_w, work=f.tile_w, waves=4, dtype=dt, **kw)


def check(dfb, f, frag):
    bg = (0.3, 0.2, 0.1, 0.9)
    cfg = config(dfb, f, background=bg, flags=dfb.DFB_KEEP_FINISHED | dfb.DFB_KEEP_SORT_ORDER)
    with dfb.Compositor(cfg, stream_handle()) as c:
        c.set_fragments(frag, f.frag.shape[0], f.layers, f.expected)
        c.composite()
        got, order = c.read(dfb.DFB_BUF_FINISHED_F32), c.read(dfb.DFB_BUF_SORT_ORDER)
    ref = oracle.composite(f.frag, f.layers, f.width, f.height, f.tile_w, f.tile_h, expected=f.expected,
                           background=bg, want_mag=True, want_order=True)
    assert_colour(got, ref["rgba"], ref["mag"], f.name)
    tiles = np.arange(f.n_tiles)
    for t, g in zip(tiles, order_as_sources(order, f.layers, tiles, f.expected, f.P)):
        assert np.array_equal(g, ref["order"][t, :, :int(f.expected[t])]), "order of tile %d" % t


@pytest.mark.parametrize("ties", [False, True])
@pytest.mark.parametrize("dtype", [np.float32, np.float16])
@pytest.mark.parametrize("tile", [20, 9, 32])
@pytest.mark.parametrize("deepest", [128, 256, 512, 513])
def test_layer_count_edges(dfb, deepest, tile, dtype, ties):
    """400 pixels a tile (a ragged last group), 81 (unaligned) and 1024."""
    counts = np.array([k for k in EDGES if k <= deepest] + [0, 5, 32], dtype=np.int32)
    f = frame_of(counts, tile, seed=deepest + tile, dtype=dtype, ties=ties)
    check(dfb, f, upload(f.frag))


@pytest.mark.parametrize("dtype", [np.float32, np.float16])
def test_misaligned_buffer(dfb, dtype):
    """Planes one element off a 4-pixel boundary."""
    torch = torch_dev()
    f = frame_of(np.array([40, 100, 300, 3]), 16, seed=5, dtype=dtype)
    buf = torch.zeros(f.frag.size + 1, dtype=torch.from_numpy(f.frag[:0]).dtype, device="cuda:0")
    buf[1:].copy_(torch.from_numpy(f.frag.reshape(-1)))
    check(dfb, f, buf[1:])


def test_accumulation_over_all_paths(dfb):
    """Three frames of tiles on every path fold into the mean, M2 and tile
    variances (the row sort keeps partial sums of its own)."""
    counts = np.array([0, 4, 32, 33, 70, 200, 512, 600], dtype=np.int32)
    f = frame_of(counts, 20, seed=9)
    wb = WelfordBound(f.n_tiles, f.P)
    mu, m2 = np.zeros((f.n_tiles, f.P, 4)), np.zeros((f.n_tiles, f.P, 3))
    with dfb.Compositor(config(dfb, f), stream_handle()) as c:
        for k in range(3):
            x = f.frag.copy()
            x[:, 0:3] *= np.float32(1 + 0.1 * k)
            c.set_fragments(upload(x), x.shape[0], f.layers, f.expected)
            c.composite(accumulate=True)
            r = oracle.composite(x, f.layers, f.width, f.height, f.tile_w, f.tile_h, expected=f.expected, want_mag=True)
            prev = mu.copy()
            oracle.accumulate(mu, m2, r["rgba"], k + 1)
            wb.step(r["rgba"], r["mag"], prev, mu, m2)
        g_mu, g_m2 = c.read(dfb.DFB_BUF_ACCUM_F32), c.read(dfb.DFB_BUF_M2_F32)
        g_var = c.read(dfb.DFB_BUF_TILE_VARIANCE)
    wb.check(g_mu, np.moveaxis(g_m2, 1, 2), mu, m2, "three frames")
    tiles = np.arange(f.n_tiles, dtype=np.int32)
    # at most 3 x 4 additions a lane, 6 over the wave and one per 32 pixels of the tile
    bound = wb.variance_bound(m2, tiles, f.width, f.height, f.tile_w, f.tile_h, 3, 12 + 6 + -(-f.P // 32))
    v = oracle.tile_variance(m2, tiles, f.width, f.height, f.tile_w, f.tile_h, 3)
    assert np.all(np.abs(g_var - v) <= bound)


def test_deep_layout_after_a_run_of_shallow_ones(dfb):
    """The queue counters of a launch come round every 64 frames: a deep
    layout, 63 frames of a layout without deep tiles, then the deep one again
    on the slot it used first."""
    deep = frame_of(np.full(24, 40), 32, seed=3)
    big = frame_of(np.full(24, 520), 8, seed=4)
    for f in (deep, big):
        shallow = frame_of(np.full(24, 2), f.tile_w, seed=6)
        a, b = upload(f.frag), upload(shallow.frag)
        with dfb.Compositor(config(dfb, f, flags=dfb.DFB_KEEP_FINISHED), stream_handle()) as c:
            c.set_fragments(a, f.frag.shape[0], f.layers, f.expected)
            c.composite()
            first = c.read(dfb.DFB_BUF_FINISHED_F32)
            c.set_fragments(b, shallow.frag.shape[0], shallow.layers, shallow.expected)
            for _ in range(63):
                c.composite()
            c.set_fragments(a, f.frag.shape[0], f.layers, f.expected)
            c.composite()
            assert np.array_equal(c.read(dfb.DFB_BUF_FINISHED_F32), first)
