"""Frames with more 32-pixel groups in tiles of more than 32 layers than the chip
holds workgroups: the row sort draws runs of groups that go over the ends of
blocks and of tiles (128, 50 and 162 groups a tile, blocks of 16), and takes
other counters' units at the end.  Every pixel against the oracle; three
accumulated copies leave the mean as it is, M2 and the variances at zero; the
entry point without allocation, which walks the whole list, the same bits."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_helpers import assert_colour, stream_handle, torch_dev, upload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [np.float32, np.float16])
@pytest.mark.parametrize("tile,n_tiles,deep", [(64, 36, 45), (40, 60, 40), (72, 20, 130)])
def test_every_group_once(tile, n_tiles, deep, dtype):
    torch = torch_dev()
    import paper_2305_07083_amd as dfb
    rng = np.random.default_rng(tile)
    counts = np.where(rng.random(n_tiles) < 0.8, rng.integers(33, deep + 1, n_tiles), rng.integers(0, 33, n_tiles))
    f = workloads.generation_frame(tile * n_tiles, tile, tile, counts.astype(np.int32), 3 + tile,
                                   depth_by_generation=False).as_dtype(dtype)
    bg = (0.3, 0.2, 0.1, 0.9)
    frag = upload(f.frag)
    cfg = dfb.make_config(f.width, f.height, tile, work=tile, waves=4, background=bg, fmt=dfb.DFB_FMT_RGBAF32,
                          dtype=dfb.DFB_F16 if dtype == np.float16 else dfb.DFB_F32)
    with dfb.Compositor(cfg, stream_handle()) as c:
        c.set_fragments(frag, f.frag.shape[0], f.layers, f.expected)
        for _ in range(3):
            c.composite(accumulate=True)
        mean, m2 = c.read(dfb.DFB_BUF_ACCUM_F32), c.read(dfb.DFB_BUF_M2_F32)
        var = c.read(dfb.DFB_BUF_TILE_VARIANCE)
    assert not m2.any() and not var.any()
    ref = oracle.composite(f.frag, f.layers, f.width, f.height, tile, tile, expected=f.expected, background=bg,
                           want_mag=True)
    assert_colour(mean, ref["rgba"], ref["mag"], "%d px tiles" % tile)
    off, layer_off, kmax = dfb.layer_tables(f.layers, f.n_tiles, f.P)
    out = torch.zeros((f.n_tiles, f.P, 4), dtype=torch.float32, device="cuda:0")
    dfb.dfb_composite_noalloc(cfg, frag, torch.from_numpy(off).cuda(), torch.from_numpy(layer_off).cuda(), kmax, out,
                              stream=stream_handle())
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy().reshape(mean.shape), mean)
