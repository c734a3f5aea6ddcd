"""The correlator's two kernels at the edges of their ranges (GPU).

A time chunk of at most 768 samples (2,048 in the halves geometry) runs on the int8
kernel, a longer one on the 6-bit kernel, whose float32 sums are turned into
integers at least every 24,576 samples.  A handle with almost no workspace
keeps a frame in one chunk, so the frame's length selects the kernel; the
default handle cuts it into short chunks that are merged.  Inputs cover the
edges of the 32-input tiles and the 128-input groups, ragged counts, frames
that end within a dword and frames that start at any byte.  Sums are integers
and must equal the oracle bit for bit.
"""

import numpy as np
import pytest

import oracle
from paper_1503_06189_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def xe():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1503_06189_amd import xengine
    xengine.lib()   # fails loudly if the library is missing
    return xengine


@pytest.fixture(scope="module")
def orc():
    return oracle.load()


@pytest.fixture(scope="module")
def handles(xe):
    out = {(g, c): xe.Handle(0, workspace_bytes=0 if c == "chunked" else 256)
           for g in ("super", "halves") for c in ("one", "chunked")}
    for (g, _), h in out.items():
        h.set_geometry(g)
    yield out
    for h in out.values():
        h.close()


def _at_byte(a, offset):
    """The frame on the device, `offset` bytes past an aligned address and
    nothing of its own behind it."""
    buf = torch.empty(a.size + offset, dtype=torch.uint8, device="cuda")
    buf[offset:] = torch.from_numpy(np.ascontiguousarray(a).ravel()).cuda()
    return buf[offset:].view(a.shape)


def _check(xe, orc, h, packed, mask, B, offset, what):
    p = _at_byte(packed, offset)
    m = None if mask is None else torch.from_numpy(mask).cuda()
    print(what, flush=True)
    ev, en = orc.correlate(packed, mask, B)
    vis, cnt = xe.correlate_frame(p, m, B, handle=h)          # overwrites
    assert np.array_equal(vis.cpu().numpy().astype(np.int64), ev), what
    assert np.array_equal(cnt.cpu().numpy(), en), what
    xe.accumulate(p, m, B, vis, cnt, handle=h)
    assert np.array_equal(vis.cpu().numpy().astype(np.int64), 2 * ev), what
    assert np.array_equal(cnt.cpu().numpy(), 2 * en), what


@pytest.mark.parametrize("chunks", ["one", "chunked"])
@pytest.mark.parametrize("N", [1, 2, 3, 5, 31, 33, 126, 127, 128, 129, 130, 250, 255, 256, 257,
                               301])
def test_both_kernels_at_their_edges(xe, orc, handles, N, chunks):
    rng = np.random.default_rng(900 + N)
    lengths = [1, 63, 64, 65, 768, 769, 900, 2048, 2049] if N <= 128 else [1, 65, 768, 769, 1000]
    for k, T in enumerate(lengths):
        for F in (1, 3):
            B = (256, 100, 7)[k % 3]
            packed = rng.integers(0, 256, (T, F, N), dtype=np.uint8)
            mask = synth.bernoulli_mask(rng, F, T, B, 0.15) if k % 2 else None
            for g in ("super", "halves") if N <= 128 else ("super",):
                off = (k + F) % 4
                _check(xe, orc, handles[g, chunks], packed, mask, B, off,
                       f"{g} {chunks} N={N} F={F} T={T} B={B} offset={off}")


@pytest.mark.parametrize("geom", ["super", "halves"])
def test_sums_stay_exact_over_a_long_chunk(xe, orc, handles, geom):
    """Extreme samples (both components at 15 or 0 of the packed range) over
    a chunk of more than two segments of 24,576 samples."""
    N, F, T, B = 6, 1, 2 * 24576 + 77, 1000
    rng = np.random.default_rng(31)
    packed = rng.choice(np.array([0x00, 0x0f, 0xf0, 0xff], np.uint8), (T, F, N))
    packed[:, :, 0] = 0xff
    packed[:, :, 1] = 0xff
    packed[:, :, 2] = 0x00
    packed[:, :, 3] = 0xf0
    mask = np.zeros((F, -(-T // B)), np.uint8)
    mask[0, 24:26] = 1
    _check(xe, orc, handles[geom, "one"], packed, mask, B, 1, f"{geom} T={T}")


def test_all_lost_and_nothing_valid(xe, orc, handles):
    for N, T in ((40, 100), (40, 3000), (200, 100), (200, 3000)):
        packed = np.full((T, 2, N), 0xa5, np.uint8)
        mask = np.ones((2, -(-T // 64)), np.uint8)
        _check(xe, orc, handles["halves", "one"], packed, mask, 64, 0, f"lost N={N} T={T}")
