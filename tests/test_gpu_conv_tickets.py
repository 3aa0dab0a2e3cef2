"""The persistent convolutions hand out tiles by tickets where an XCD has more
than two tiles for each of its workgroups, from counters that every launch
leaves at zero.  With 256 compute units and at most three workgroups on each,
that is from 1537 tiles on (8 or 16 rows of 32 pixels): ten images of 640 x 1024
have 1600 or more at each of the three resolutions.  Sizes with and without tickets
in turn, the outputs cleared in between: always the same bits."""
import numpy as np
import pytest

import workloads
from gpu_helpers import stream_handle, torch_dev, upload

pytestmark = pytest.mark.gpu


def test_forwards_with_and_without_tickets():
    """Ten images at once, against each image alone and a small forward in
    between: the same bits, three times over."""
    torch = torch_dev()
    import paper_2305_07083_amd as dfb
    n, h, w = 10, 640, 1024
    gen = torch.Generator(device="cuda").manual_seed(4)
    x = torch.rand((n, h, w, 6), generator=gen, device="cuda")
    small = torch.rand((1, 64, 128, 6), generator=gen, device="cuda")
    out, one, tiny = (torch.empty(s + (3,), device="cuda") for s in ((n, h, w), (1, h, w), (1, 64, 128)))
    with dfb.Denoiser(n * h * w, seed=5, stream=stream_handle()) as d:
        dfb.dfb_denoiser_forward(d.net, small, tiny, 1, 64, 128)
        first_tiny = tiny.clone()
        first = None
        for _ in range(3):
            out.fill_(-1)
            dfb.dfb_denoiser_forward(d.net, x, out, n, h, w)
            if first is None:
                first = out.clone()
            assert torch.equal(out, first)
            tiny.fill_(-1)
            dfb.dfb_denoiser_forward(d.net, small, tiny, 1, 64, 128)
            assert torch.equal(tiny, first_tiny)
        for i in range(n):
            one.fill_(-1)
            dfb.dfb_denoiser_forward(d.net, x[i].contiguous(), one, 1, h, w)
            assert torch.equal(one[0], first[i]), i


@pytest.mark.parametrize("W,H", [(1024, 1028), (2048, 1024)])
def test_frames_denoised_in_turn(W, H):
    """dfb_denoise, whose first and last layers read and write the frame: two
    frames and a small one in turn through one network, the denoised buffer
    of each overwritten by the other accumulation's in between; RGB as
    dfb_denoiser_forward gives it on the frame's own input."""
    torch = torch_dev()
    import paper_2305_07083_amd as dfb
    comps, want = [], []
    with dfb.Denoiser(W * H, seed=6, stream=stream_handle()) as d:
        for i, (cw, ch) in enumerate([(W, H), (W, H), (64, 64)]):
            f = workloads.brick_frame(cw, ch, (2, 2, 2), 64, seed=31 + i)
            cfg = dfb.make_config(cw, ch, 64, work=32, waves=4)
            c = dfb.Compositor(cfg, stream_handle())
            frags = [upload(workloads.noisy_colour(f, 0.2, 4, k)) for k in range(2)]
            comps.append((c, f, frags))
        def state(i, n):  # n frames in compositor i's accumulation
            c, f, frags = comps[i]
            c.reset()
            for k in range(n):
                c.set_fragments(frags[k], f.frag.shape[0], f.layers, f.expected)
                c.composite(accumulate=True)
            return c
        got = {}
        for turn in range(3):
            for n in (1, 2):
                for i, (cw, ch) in enumerate([(W, H), (W, H), (64, 64)]):
                    c = state(i, n)
                    dfb.dfb_denoise(c.h, d.net, 1e30)
                    y = c.read(dfb.DFB_BUF_DENOISED_F32)
                    if turn == 0:
                        got[i, n] = y
                        inp = torch.empty((ch, cw, 6), dtype=torch.float32, device="cuda")
                        dfb.dfb_denoiser_frame_input(c.h, inp)
                        out = torch.empty((1, ch, cw, 3), dtype=torch.float32, device="cuda")
                        dfb.dfb_denoiser_forward(d.net, inp, out, 1, ch, cw)
                        q, tx = np.arange(64 * 64), -(-cw // 64)
                        t = np.arange(y.shape[0])[:, None]
                        xs, ys = (t % tx) * 64 + q % 64, (t // tx) * 64 + q // 64
                        inside = (xs < cw) & (ys < ch)
                        np.testing.assert_allclose(y[inside][:, :3], out.cpu().numpy()[0][ys[inside], xs[inside]], rtol=0,
                                                   atol=1e-6)
                    assert np.array_equal(y, got[i, n]), (turn, n, i)
        assert not np.array_equal(got[0, 1], got[0, 2]) and not np.array_equal(got[0, 1], got[1, 1])
    for c, _, _ in comps:
        c.close()
