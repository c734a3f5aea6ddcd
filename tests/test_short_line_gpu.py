"""Frames of one chunk on either side of the lines between the int8 and the 6-bit
kernel of the super geometry: 24, 32 and 40 steps of 32 samples (GPU).  Sums are
integers and must equal the oracle.
"""

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def handle():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1503_06189_amd import xengine
    h = xengine.Handle(0, workspace_bytes=256)     # frames stay in one chunk
    yield h
    h.close()


@pytest.mark.parametrize("N,steps", [(130, 40), (132, 40), (192, 40), (255, 32), (256, 32),
                                     (257, 24), (260, 40), (388, 32), (520, 40), (772, 24)])
@pytest.mark.parametrize("offset", [0, 1])
def test_both_sides(handle, N, steps, offset):
    from paper_1503_06189_amd import xengine as xe
    F = 2 if N < 300 else 1
    g = torch.Generator(device="cuda")
    g.manual_seed(N)
    for line in sorted({24, steps}):
        for T in (32 * line - 31, 32 * line, 32 * line + 1):
            print(f"line N={N} T={T} offset={offset}", flush=True)
            B = 48
            buf = torch.randint(0, 256, (T * F * N + offset,), dtype=torch.uint8, device="cuda",
                                generator=g)
            packed = buf[offset:].view(T, F, N)
            mask = (torch.rand((F, -(-T // B)), device="cuda", generator=g) < 0.2).to(torch.uint8)
            vis, count = xe.correlate_frame(packed, mask, B, handle=handle)
            xe.accumulate(packed, mask, B, vis, count, handle=handle)
            want, n = oracle.load().correlate(packed.cpu().numpy(), mask.cpu().numpy(), B)
            assert np.array_equal(count.cpu().numpy(), 2 * n)
            assert np.array_equal(vis.cpu().numpy().astype(np.int64), 2 * want)
