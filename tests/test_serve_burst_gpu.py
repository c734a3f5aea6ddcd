"""Frames offered all at once share the first launch (GPU).

The frames are large, so that a copy takes longer than the launch that consumes
it: served as they land, every slice would go out alone.
"""

import numpy as np
import pytest

import oracle
from paper_1503_06189_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def burst():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    specs = [synth.StreamSpec(k, 64, 64, 4096, 1, 0.02, 6.4e9, 4000 + k) for k in range(4)]
    return specs, {s.stream_id: [synth.stream_frame(s, 0, 256)] for s in specs}


# whole frames; slices; a pool of three slots, which as many streams share
@pytest.mark.parametrize("kw,first", [({}, 4), ({"slice_samples": 1024}, 4),
                                      ({"slot_bytes": 16 << 20, "pool_bytes": 3 * ((16 << 20) + 4096)}, 3)])
def test_first_launch_takes_a_slice_of_every_stream(burst, kw, first):
    from paper_1503_06189_amd import serve
    specs, pool = burst
    orc = oracle.load()
    serve.run_load(specs, speed=float("inf"), pool=pool)      # (kernels loaded)
    res = serve.run_load(specs, speed=float("inf"), pool=pool, **kw)
    print(f"burst {kw}: batches {res.server.batch_sizes}", flush=True)
    assert res.server.batch_sizes[0] == first
    assert res.stats["mean_batch"] > 1.0
    assert sorted(res.server.results) == [s.stream_id for s in specs]
    for s in specs:
        fr = pool[s.stream_id][0]
        vis, count = orc.correlate(fr.packed, fr.mask, fr.B)
        (r,) = res.server.results[s.stream_id]
        assert np.array_equal(r.count, count) and np.array_equal(r.vis.astype(np.int64), vis)
