"""Frames whose tiles all have more than 32 layers: the frame's last launch,
which counts its workgroups, recycles the counters' slots and advances the
frame state, then has no unit of its own.  More frames in a row than three
times around the counters' 64 slots, from two fragment buffers in turn, so that
a unit left out or a stale frame shows; the first two against the oracle, every
later one the same bits, the frames counted exactly."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_helpers import assert_colour, stream_handle, torch_dev, upload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("low,high,tile,n_tiles,shift", [
    (33, 60, 32, 24, 0),     # the row sort alone
    (33, 60, 16, 900, 0),    # by tickets
    (513, 530, 8, 24, 0),    # the LDS sort alone
    (500, 530, 8, 24, 0),    # both
    (33, 60, 16, 24, 1),     # planes off a 4-pixel boundary: the LDS sort
])
@pytest.mark.parametrize("waves", [1, 4])
def test_frames_without_shallow_tiles(low, high, tile, n_tiles, shift, waves):
    torch = torch_dev()
    import paper_2305_07083_amd as dfb
    counts = np.random.default_rng(tile + n_tiles).integers(low, high + 1, n_tiles).astype(np.int32)
    f = workloads.generation_frame(tile * n_tiles, tile, tile, counts, 11, depth_by_generation=False)
    bg = (0.3, 0.2, 0.1, 0.9)
    frags, firsts = [], []
    for k in range(2):
        x = f.frag.copy()
        x[:, 0:3] *= np.float32(1 - 0.5 * k)
        buf = torch.zeros(x.size + shift, dtype=torch.float32, device="cuda:0")
        buf[shift:].copy_(upload(x).reshape(-1))
        frags.append(buf[shift:])
        ref = oracle.composite(x, f.layers, f.width, f.height, tile, tile, expected=f.expected, background=bg, want_mag=True)
        firsts.append((ref["rgba"], ref["mag"]))
    cfg = dfb.make_config(f.width, f.height, tile, work=tile, waves=waves, background=bg, fmt=dfb.DFB_FMT_RGBAF32)
    out = torch.empty((2, f.n_tiles, f.P, 4), dtype=torch.float32, device="cuda:0")
    got = torch.empty_like(out[0])
    same = torch.ones((), dtype=torch.bool, device="cuda:0")
    with dfb.Compositor(cfg, stream_handle()) as c:
        for k in range(200):
            c.set_fragments(frags[k % 2], f.frag.shape[0], f.layers, f.expected)
            c.composite()
            dfb.dfb_read_tiles(c.h, dfb.DFB_BUF_FINAL, 0, f.n_tiles, out[k] if k < 2 else got, True)
            if k >= 2:
                same &= (got == out[k % 2]).all()
        assert bool(same)
        for k in range(130):
            c.composite(accumulate=True)
        assert c.info().accumulation_id == 130
    for k in range(2):
        assert_colour(out[k].cpu().numpy().reshape(firsts[k][0].shape), *firsts[k], "buffer %d" % k)
