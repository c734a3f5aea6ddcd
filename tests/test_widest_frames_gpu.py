"""The widest frames that the ABI accepts (F * N up to XE_MAX_FN), on the GPU.

Such a frame runs in one chunk of at most 4 steps, and its loads reach as far
as byte offsets may.  The channels compared with the oracle are the first, the
last and some between.
"""

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

WIDEST = 4194304


@pytest.fixture(scope="module")
def xe():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1503_06189_amd import xengine
    xengine.lib()
    return xengine


# one input, unaligned rows, the halves and the super geometry; a batch runs
# the 6-bit kernel whatever the length
@pytest.mark.parametrize("N,F,T,batch", [(1, WIDEST, 100, False), (1, WIDEST - 1, 128, False),
                                         (8, 524288, 128, False), (127, 33026, 61, False),
                                         (129, 32513, 40, False), (132, 31775, 128, False),
                                         (32, 131072, 128, True)])
def test_widest_frames(xe, N, F, T, batch):
    print(f"widest N={N} F={F} T={T} batch={batch}", flush=True)
    B = 16
    g = torch.Generator(device="cuda")
    g.manual_seed(N + T)
    packed = torch.randint(0, 256, (T, F, N), dtype=torch.uint8, device="cuda", generator=g)
    mask = (torch.rand((F, -(-T // B)), device="cuda", generator=g) < 0.1).to(torch.uint8)
    vis, count = xe.new_accumulators(N, F)
    if batch:
        xe.accumulate_batch([(packed, mask, B, vis, count)])
    else:
        xe.accumulate(packed, mask, B, vis, count)
    some = torch.tensor(sorted({0, 1, F // 3, F // 2, F - 2, F - 1}), device="cuda")
    want, n = oracle.load().correlate(packed[:, some].contiguous().cpu().numpy(),
                                      mask[some].contiguous().cpu().numpy(), B)
    assert np.array_equal(count[some].cpu().numpy(), n)
    assert np.array_equal(vis[some].cpu().numpy().astype(np.int64), want)
