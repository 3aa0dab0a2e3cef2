"""The row sort's keys at the special depths: NaNs of either sign and any
payload (after every number, equal among themselves), both zeros (equal), both
infinities, subnormals, the largest and smallest numbers, and runs of equal
depths, where the source id decides.  Order bit-exact against the oracle."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_helpers import order_as_sources, stream_handle, torch_dev, upload

pytestmark = pytest.mark.gpu


def special_depths(dtype):
    if dtype == np.float16:
        bits = np.array([0x0000, 0x8000, 0x7C00, 0xFC00, 0x7E00, 0xFE01, 0x7C01, 0xFFFF, 0x0001, 0x8001, 0x03FF, 0x7BFF,
                         0xFBFF, 0x3C00, 0xBC00, 0x3C01], dtype=np.uint16)
    else:
        bits = np.array([0x00000000, 0x80000000, 0x7F800000, 0xFF800000, 0x7FC00000, 0xFFC00001, 0x7F800001, 0xFFFFFFFF,
                         0x00000001, 0x80000001, 0x007FFFFF, 0x7F7FFFFF, 0xFF7FFFFF, 0x3F800000, 0xBF800000, 0x3F800001],
                        dtype=np.uint32)
    return bits.view(dtype)


@pytest.mark.parametrize("dtype", [np.float32, np.float16])
@pytest.mark.parametrize("deepest", [128, 512])
def test_special_depths(deepest, dtype):
    torch_dev()
    import paper_2305_07083_amd as dfb
    counts = np.array([33, 64, 80, 128] + ([190, 256, 384, 512] if deepest == 512 else []), dtype=np.int32)
    f = workloads.generation_frame(16 * len(counts), 16, 16, counts, 17, depth_by_generation=False).as_dtype(dtype)
    rng = np.random.default_rng(deepest)
    pick = rng.random(f.frag[:, 4].shape) < 0.6
    depth = np.where(pick, special_depths(dtype)[rng.integers(0, 16, pick.shape)], f.frag[:, 4])
    f.frag[:, 4] = depth
    cfg = dfb.make_config(f.width, f.height, 16, work=16, waves=4, flags=dfb.DFB_KEEP_SORT_ORDER,
                          dtype=dfb.DFB_F16 if dtype == np.float16 else dfb.DFB_F32)
    with dfb.Compositor(cfg, stream_handle()) as c:
        c.set_fragments(upload(f.frag), f.frag.shape[0], f.layers, f.expected)
        c.composite()
        order = c.read(dfb.DFB_BUF_SORT_ORDER)
    ref = oracle.composite(f.frag, f.layers, f.width, f.height, 16, 16, expected=f.expected, want_order=True)
    tiles = np.arange(f.n_tiles)
    for t, g in zip(tiles, order_as_sources(order, f.layers, tiles, f.expected, f.P)):
        assert np.array_equal(g, ref["order"][t, :, :int(f.expected[t])]), "order of tile %d" % t
