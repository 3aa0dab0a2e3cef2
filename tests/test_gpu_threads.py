"""Handles of several host threads, each on a stream of its own: their first
frames choose launch shapes at the same time and enter them into the cache that
all handles share; every frame against the oracle."""
import threading

import numpy as np
import pytest

import oracle
import workloads
from gpu_helpers import assert_colour, torch_dev, upload

pytestmark = pytest.mark.gpu

BG = (0.3, 0.2, 0.1, 0.9)


def test_handles_on_threads():
    torch = torch_dev()
    import paper_2305_07083_amd as dfb
    jobs = []
    for i in range(6):
        counts = np.random.default_rng(i).integers(0, (8, 16, 30, 45, 100, 140)[i], 9 + i).astype(np.int32)
        f = workloads.generation_frame(32 * len(counts), 32, 32, counts, 60 + i, depth_by_generation=False)
        jobs.append((f, upload(f.frag), torch.cuda.Stream()))
    torch.cuda.synchronize()
    got, errors = {}, []

    def work(i):
        f, frag, s = jobs[i]
        try:
            for turn in range(3):  # the second and third handle find the first one's shape
                cfg = dfb.make_config(f.width, f.height, 32, background=BG, fmt=dfb.DFB_FMT_RGBAF32)
                with dfb.Compositor(cfg, s.cuda_stream) as c:
                    c.set_fragments(frag, f.frag.shape[0], f.layers, f.expected)
                    for _ in range(20):
                        c.composite()
                    got[i, turn] = c.read(dfb.DFB_BUF_FINAL)
        except Exception as e:  # shown by the test's own thread
            errors.append((i, e))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(jobs))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for i, (f, _, _) in enumerate(jobs):
        ref = oracle.composite(f.frag, f.layers, f.width, f.height, 32, 32, expected=f.expected, background=BG, want_mag=True)
        for turn in range(3):
            assert_colour(got[i, turn], ref["rgba"], ref["mag"], "thread %d" % i)
