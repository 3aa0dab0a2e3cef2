"""Graphs that the caller captured on a handle, replayed after the handle took
other layer layouts: what they point to (partial sums of the variance, the
layout's tables) has to stay where it was."""
import numpy as np
import pytest

import workloads
from gpu_helpers import torch_dev, upload

pytestmark = pytest.mark.gpu

BUFS = ("ACCUM_F32", "M2_F32", "TILE_VARIANCE", "FINAL")


@pytest.fixture(scope="module")
def dfb():
    torch_dev()
    import paper_2305_07083_amd as m
    m.load()
    return m


def frame(counts, seed):
    return workloads.generation_frame(64 * len(counts), 64, 64, np.asarray(counts, dtype=np.int32), seed,
                                      depth_by_generation=False)


def scaled(f, k):
    x = f.frag.copy()
    x[:, 0:3] *= np.float32(1 - 0.1 * k)
    return x


@pytest.mark.parametrize("work", [(32, 32), None])
def test_accumulating_graph_after_a_deep_layout(dfb, work):
    """A captured accumulating frame of shallow tiles, replayed after the
    handle's first layout of deep ones: mean, M2, variances and display as
    without a graph, bit for bit."""
    torch = torch_dev()
    a, b = frame([3, 0, 7, 20, 1, 30], 1), frame([3, 40, 7, 120, 1, 33], 2)
    s = torch.cuda.Stream()
    buf = torch.empty(a.frag.shape, dtype=torch.float32, device="cuda:0")
    deep = upload(b.frag)
    torch.cuda.synchronize()
    kw = dict(work=work[0], waves=2) if work else {}
    cfg = dfb.make_config(a.width, a.height, 64, fmt=dfb.DFB_FMT_RGBA8, **kw)
    with torch.cuda.stream(s), dfb.Compositor(cfg, s.cuda_stream) as d, dfb.Compositor(cfg, s.cuda_stream) as g:
        buf.copy_(torch.from_numpy(scaled(a, 0)))
        for c in (d, g):
            c.set_fragments(buf, a.frag.shape[0], a.layers, a.expected)
            c.composite(accumulate=True)
        s.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            g.composite(accumulate=True)
        for c in (d, g):
            c.set_fragments(deep, b.frag.shape[0], b.layers, b.expected)
            c.composite()
            c.composite(accumulate=True)
        d.set_fragments(buf, a.frag.shape[0], a.layers, a.expected)
        for k in range(1, 5):
            buf.copy_(torch.from_numpy(scaled(a, k)))
            d.composite(accumulate=True)
            graph.replay()
            s.synchronize()
            for n in BUFS:
                x, y = (c.read(getattr(dfb, "DFB_BUF_" + n)) for c in (d, g))
                assert x.tobytes() == y.tobytes(), "%s after replay %d" % (n, k)
        assert g.info().accumulation_id == d.info().accumulation_id == 6


def test_graph_after_two_layouts(dfb):
    """Two sets of tables take turns, so the second new layout is written over
    the one a graph was captured with: with no more layers than that one, at
    the same addresses, so replays composite it."""
    torch = torch_dev()
    a, b = frame([3, 0, 7, 8, 1, 5], 3), frame([1, 2, 3, 4, 5, 6], 4)
    keep = np.arange(len(a.layers)) % 3 != 1  # the third layout: some of the first one's layers
    fewer = np.ascontiguousarray(a.layers[keep])
    s = torch.cuda.Stream()
    fa, fb = upload(a.frag), upload(b.frag)
    torch.cuda.synchronize()
    cfg = dfb.make_config(a.width, a.height, 64, work=32, waves=2, fmt=dfb.DFB_FMT_RGBAF32)
    with torch.cuda.stream(s), dfb.Compositor(cfg, s.cuda_stream) as alone, dfb.Compositor(cfg, s.cuda_stream) as g:
        alone.set_fragments(fa, a.frag.shape[0], fewer)
        alone.composite()
        want = alone.read(dfb.DFB_BUF_FINAL)
        g.set_fragments(fa, a.frag.shape[0], a.layers, a.expected)
        g.composite()
        first = g.read(dfb.DFB_BUF_FINAL)
        s.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            g.composite()
        g.set_fragments(fb, b.frag.shape[0], b.layers, b.expected)
        g.composite()
        graph.replay()
        s.synchronize()
        assert np.array_equal(g.read(dfb.DFB_BUF_FINAL), first)
        g.set_fragments(fa, a.frag.shape[0], fewer)
        g.composite()
        assert np.array_equal(g.read(dfb.DFB_BUF_FINAL), want)
        g.set_fragments(fb, b.frag.shape[0], b.layers, b.expected)
        g.composite()
        for _ in range(3):
            graph.replay()
            s.synchronize()
            assert np.array_equal(g.read(dfb.DFB_BUF_FINAL), want)
