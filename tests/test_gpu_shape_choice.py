"""Which frames choose a launch shape.  Choosing times every candidate (15 shapes
of 64x64 tiles, 10 frames each, with a synchronisation after each), so a frame that
chooses takes over 100 times as long as one that does not, and one that does not
a few times as long at most: 20 separates them."""
import time

import numpy as np
import pytest

import oracle
import workloads
from gpu_helpers import assert_colour, stream_handle, torch_dev, upload

pytestmark = pytest.mark.gpu

BG = (0.3, 0.2, 0.1, 0.9)


def timed(dfb, c):
    dfb.dfb_synchronize(c.h)
    t = time.perf_counter()
    c.composite()
    dfb.dfb_synchronize(c.h)
    return time.perf_counter() - t


def chooses(dfb, c):
    """Whether the next frame chooses a shape: its time against the frames after it."""
    first = timed(dfb, c)
    return first > 20 * min(timed(dfb, c) for _ in range(5))


def frame(counts, seed, tile=64):
    counts = np.asarray(counts, dtype=np.int32)
    return workloads.generation_frame(tile * len(counts), tile, tile, counts, seed, depth_by_generation=False)


def check(dfb, c, f):
    ref = oracle.composite(f.frag, f.layers, f.width, f.height, f.tile_w, f.tile_h, expected=f.expected, background=BG,
                           want_mag=True)
    assert_colour(c.read(dfb.DFB_BUF_FINAL), ref["rgba"], ref["mag"], f.name)


def test_frames_of_deep_tiles_alone_choose_nothing():
    """With every tile in the row sort's launch, whose shape is fixed, there is
    nothing to choose from; the first frame of the same class of layer counts
    that has other tiles chooses, in this handle and in the next, and the choice
    is kept."""
    torch_dev()
    import paper_2305_07083_amd as dfb
    deep, mixed = frame([40, 50, 60, 64], 1), frame([40, 3, 60, 9], 2)
    cfg = dfb.make_config(deep.width, deep.height, 64, background=BG, fmt=dfb.DFB_FMT_RGBAF32)
    fd, fm = upload(deep.frag), upload(mixed.frag)
    with dfb.Compositor(cfg, stream_handle()) as warm:  # kernels loaded, another class of layer counts
        few = frame([3, 40, 100, 7], 3)
        warm.set_fragments(upload(few.frag), few.frag.shape[0], few.layers, few.expected)
        warm.composite()
        dfb.dfb_synchronize(warm.h)
    with dfb.Compositor(cfg, stream_handle()) as c:
        c.set_fragments(fd, deep.frag.shape[0], deep.layers, deep.expected)
        assert not chooses(dfb, c)
        check(dfb, c, deep)
        c.set_fragments(fm, mixed.frag.shape[0], mixed.layers, mixed.expected)
        assert chooses(dfb, c)
        check(dfb, c, mixed)
        shape = (c.info().work_w, c.info().work_h, c.info().waves_per_tile)
        for f, d in ((deep, fd), (mixed, fm)) * 2:
            c.set_fragments(d, f.frag.shape[0], f.layers, f.expected)
            assert not chooses(dfb, c)
            check(dfb, c, f)
            assert shape == (c.info().work_w, c.info().work_h, c.info().waves_per_tile)
    with dfb.Compositor(cfg, stream_handle()) as c:  # from the cache
        c.set_fragments(fm, mixed.frag.shape[0], mixed.layers, mixed.expected)
        c.composite()
        assert shape == (c.info().work_w, c.info().work_h, c.info().waves_per_tile)


def test_stand_in_under_capture():
    """A layout that would choose is captured with the shape at hand."""
    torch = torch_dev()
    import paper_2305_07083_amd as dfb
    deep, mixed = frame([70, 80, 90, 128], 4), frame([70, 3, 90, 9], 5)
    cfg = dfb.make_config(deep.width, deep.height, 64, background=BG, fmt=dfb.DFB_FMT_RGBAF32)
    fd, fm = upload(deep.frag), upload(mixed.frag)
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    with torch.cuda.stream(s), dfb.Compositor(cfg, s.cuda_stream) as c:
        c.set_fragments(fd, deep.frag.shape[0], deep.layers, deep.expected)
        c.composite()
        c.set_fragments(fm, mixed.frag.shape[0], mixed.layers, mixed.expected)
        s.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            c.composite()
        for _ in range(3):
            graph.replay()
            s.synchronize()
            check(dfb, c, mixed)
        c.composite()
        check(dfb, c, mixed)


@pytest.mark.parametrize("dtype", [np.float32, np.float16])
def test_buffers_of_both_alignments(dtype):
    """Planes off a 4-pixel boundary send the tiles of more than 32 layers to
    the LDS sort, whose time depends on the shape: such a buffer's first frame
    chooses for itself (or takes the choice from the cache), then buffers of both
    kinds in turn choose nothing, launched or replayed, each with its own result
    and its own shape, and under capture the shape at hand is used."""
    torch = torch_dev()
    import paper_2305_07083_amd as dfb
    f = frame([40, 3, 60, 9, 64, 33, 35], 6 + np.dtype(dtype).itemsize).as_dtype(dtype)
    cfg = dfb.make_config(f.width, f.height, 64, background=BG, fmt=dfb.DFB_FMT_RGBAF32,
                          dtype=dfb.DFB_F16 if dtype == np.float16 else dfb.DFB_F32)
    n = f.frag.size
    raw = torch.zeros(n + 1, dtype=torch.from_numpy(f.frag[:0]).dtype, device="cuda:0")
    bufs = [upload(f.frag), raw[1:]]
    raw[1:].copy_(bufs[0].reshape(-1))
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    with torch.cuda.stream(s), dfb.Compositor(cfg, s.cuda_stream) as c:
        shapes = []
        for d in bufs:
            c.set_fragments(d, f.frag.shape[0], f.layers, f.expected)
            assert chooses(dfb, c)
            check(dfb, c, f)
            shapes.append((c.info().work_w, c.info().work_h, c.info().waves_per_tile))
        for replay in (False, True):
            for k in range(6):
                c.set_fragments(bufs[k % 2], f.frag.shape[0], f.layers, f.expected)
                if replay:
                    c.composite(replay=True)
                else:
                    assert not chooses(dfb, c)
                    assert shapes[k % 2] == (c.info().work_w, c.info().work_h, c.info().waves_per_tile)
                check(dfb, c, f)
        c.set_fragments(bufs[0], f.frag.shape[0], f.layers, f.expected)
        c.composite()
        c.set_fragments(bufs[1], f.frag.shape[0], f.layers, f.expected)
        s.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            c.composite()
        for _ in range(3):
            graph.replay()
            s.synchronize()
            check(dfb, c, f)
    with dfb.Compositor(cfg, stream_handle()) as c:  # each from the cache
        for k in (1, 0, 1):
            c.set_fragments(bufs[k], f.frag.shape[0], f.layers, f.expected)
            c.composite()
            assert shapes[k] == (c.info().work_w, c.info().work_h, c.info().waves_per_tile)
            check(dfb, c, f)


def test_fixed_units_captured_first():
    """With the work unit and the waves given, a buffer off a 4-pixel boundary
    leaves only the LDS sort's budget to choose (from 129 layers on); captured
    before any frame, it takes the aligned buffer's."""
    torch = torch_dev()
    import paper_2305_07083_amd as dfb
    f = frame([150, 3, 200, 40], 9, tile=32)
    cfg = dfb.make_config(f.width, f.height, 32, work=32, waves=4, background=BG, fmt=dfb.DFB_FMT_RGBAF32)
    raw = torch.zeros(f.frag.size + 1, dtype=torch.float32, device="cuda:0")
    raw[1:].copy_(upload(f.frag).reshape(-1))
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    with torch.cuda.stream(s), dfb.Compositor(cfg, s.cuda_stream) as c:
        c.set_fragments(raw[1:], f.frag.shape[0], f.layers, f.expected)
        s.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            c.composite()
        for _ in range(3):
            graph.replay()
            s.synchronize()
            check(dfb, c, f)
        c.composite()
        check(dfb, c, f)
