"""The work queue of a frame launch: frames whose units each get a workgroup
of their own (no tickets), frames that go through the tickets, and few blocks
of units over few counters, for more frames in a row than a counter has slots.
Every frame must cover every unit exactly once: identical frames leave the
running mean bit-identical to the first and M2 at zero."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_helpers import assert_colour, stream_handle, torch_dev, upload

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dfb():
    torch_dev()
    import paper_2305_07083_amd as m
    m.load()
    return m


@pytest.mark.parametrize("n_tiles,tile,work,waves", [
    (1, 16, 16, 1),       # one unit
    (1, 64, 16, 4),       # one block of 16 units
    (17, 32, 16, 2),      # 17 blocks over 16 counters
    (40, 16, 16, 4),
    (256, 32, 16, 4),     # 1024 workgroups
    (2304, 16, 16, 4),    # about as many units as the chip holds workgroups
    (700, 64, 16, 4),     # 11200 units
    (9000, 16, 16, 1),
])
@pytest.mark.parametrize("op", [0, 2])
def test_every_unit_once(dfb, n_tiles, tile, work, waves, op):
    counts = np.arange(n_tiles, dtype=np.int32) % 4
    cols = max(d for d in range(1, 101) if n_tiles % d == 0)
    f = workloads.generation_frame(tile * cols, tile * (n_tiles // cols), tile, counts, 7 + n_tiles,
                                   depth_by_generation=False)
    frag = upload(f.frag)
    bg = (0.3, 0.2, 0.1, 0.9)
    cfg = dfb.make_config(f.width, f.height, tile, work=work, waves=waves, background=bg, op=op,
                          fmt=dfb.DFB_FMT_RGBAF32)
    with dfb.Compositor(cfg, stream_handle()) as c:
        c.set_fragments(frag, f.frag.shape[0], f.layers, f.expected)
        c.composite(accumulate=True)
        first = c.read(dfb.DFB_BUF_ACCUM_F32)
        for _ in range(132):
            c.composite(accumulate=True)
        assert c.info().accumulation_id == 133
        assert np.array_equal(c.read(dfb.DFB_BUF_ACCUM_F32), first)
        assert not c.read(dfb.DFB_BUF_M2_F32).any()
    if op == 0:
        ref = oracle.composite(f.frag, f.layers, f.width, f.height, tile, tile, expected=f.expected, background=bg,
                               want_mag=True)
        assert_colour(first, ref["rgba"], ref["mag"], "%d tiles" % n_tiles)
        torch = torch_dev()
        off, layer_off, kmax = dfb.layer_tables(f.layers, f.n_tiles, f.P)
        out = torch.zeros((f.n_tiles, f.P, 4), dtype=torch.float32, device="cuda:0")
        off, layer_off = torch.from_numpy(off).cuda(), torch.from_numpy(layer_off).cuda()
        for _ in range(2):
            dfb.dfb_composite_noalloc(cfg, frag, off, layer_off, kmax, out, stream=stream_handle())
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy(), first)


def test_layouts_of_changing_size(dfb):
    """Every frame a layout of another size, with no synchronisation between:
    the two table sets and their staging grow and are reused while earlier
    frames may still be in flight.  The last frame of each size against the
    oracle, bit-identical to the same layout on its own."""
    torch = torch_dev()
    rng = np.random.default_rng(5)
    frames = []
    for k in range(7):
        counts = rng.integers(0, 3 + 9 * (k % 4), 96).astype(np.int32)
        f = workloads.generation_frame(32 * 12, 32 * 8, 32, counts, 50 + k, depth_by_generation=False)
        frames.append((f, upload(f.frag)))
    cfg = dfb.make_config(frames[0][0].width, frames[0][0].height, 32, work=32, waves=4, fmt=dfb.DFB_FMT_RGBAF32)
    alone = []
    for f, frag in frames:
        with dfb.Compositor(cfg, stream_handle()) as c:
            c.set_fragments(frag, f.frag.shape[0], f.layers, f.expected)
            c.composite()
            alone.append(c.read(dfb.DFB_BUF_FINAL))
        ref = oracle.composite(f.frag, f.layers, f.width, f.height, 32, 32, expected=f.expected, want_mag=True)
        assert_colour(alone[-1], ref["rgba"], ref["mag"], f.name)
    with dfb.Compositor(cfg, stream_handle()) as c:
        out = [torch.empty((f.n_tiles, f.P, 4), dtype=torch.float32, device="cuda:0") for f, _ in frames * 3]
        for o, (f, frag) in zip(out, frames * 3):
            c.set_fragments(frag, f.frag.shape[0], f.layers, f.expected)
            c.composite()
            dfb.dfb_read_tiles(c.h, dfb.DFB_BUF_FINAL, 0, f.n_tiles, o, True)
        dfb.dfb_synchronize(c.h)
        for o, a in zip(out, alone * 3):
            assert np.array_equal(o.cpu().numpy().reshape(a.shape), a)
