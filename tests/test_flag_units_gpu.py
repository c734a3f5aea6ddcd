"""The two Gram kernels of the flag counts at the edges of their ranges (GPU).

Frames whose units of tiles fill the GPU up to twice over (and all of at most
256 inputs) are counted by the unit kernel, larger ones by the wide kernel; so
the number of channels selects the kernel.  Inputs cover the edges of words,
128-input groups and 256-input super blocks, lengths those of a K-step (64
samples), of a batch of every wave (2,048) and of a chunk (32,768).  Counts
must equal the oracle's, added to what the array held.
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


def _check(xe, orc, flags, mask, N, B, offset, what):
    print(what, flush=True)
    F, T, W = flags.shape
    c, d = orc.flag_counters(flags, mask, N, B)
    # `offset` words past a 16-byte boundary, nothing of its own behind
    buf = torch.empty(flags.size + offset, dtype=torch.int32, device="cuda")
    buf[offset:] = torch.from_numpy(np.ascontiguousarray(flags).view(np.int32).ravel()).cuda()
    m = None if mask is None else torch.from_numpy(mask).cuda()
    dcount = xe.new_flag_counts(N, F)
    dcount += 3
    xe.flag_accumulate(buf[offset:].view(F, T, W), m, B, N, dcount)
    got = dcount.cpu().numpy().astype(np.int64)
    assert np.array_equal(got, d + 3), what


def _flags(rng, F, T, N, kind):
    if kind == "bursts":
        return synth.fengine_flags(rng, T, F, N, 0.01, mean_run=32.0, garbage_padding=True)
    if kind == "scattered":
        return synth.random_flags(rng, T, F, N, 0.03, garbage_padding=True)
    flags = np.zeros((F, T, synth.flag_words(N)), np.uint32)
    flags[:, -1, :] = 0xffffffff          # the last sample only
    flags[:, 0, -1] = 0xffffffff          # and the last word of the first
    return flags


@pytest.mark.parametrize("N", [1, 31, 32, 33, 127, 128, 129, 255, 256, 257, 385, 512])
@pytest.mark.parametrize("kind", ["bursts", "scattered", "ends"])
def test_unit_kernel(xe, orc, N, kind):
    rng = np.random.default_rng(700 + N)
    for k, T in enumerate((1, 64, 65, 200, 2048, 2049) if N <= 256 else (1, 65, 2100)):
        F, B = 1 + k % 2, (256, 100, 3)[k % 3]
        mask = synth.bernoulli_mask(rng, F, T, B, 0.1) if k % 2 else None
        _check(xe, orc, _flags(rng, F, T, N, kind), mask, N, B, k % 4,
               f"{kind} N={N} F={F} T={T} B={B}")


@pytest.mark.parametrize("N,F", [(257, 56), (257, 57), (385, 32), (385, 33), (513, 5), (513, 6),
                                 (1000, 2), (1000, 3)])
def test_both_sides_of_the_line(xe, orc, N, F):
    rng = np.random.default_rng(800 + N + F)
    for k, kind in enumerate(("bursts", "scattered", "ends")):
        T, B = (150, 65, 33)[k], 16
        mask = synth.bernoulli_mask(rng, F, T, B, 0.1)
        _check(xe, orc, _flags(rng, F, T, N, kind), mask, N, B, 0 if N != 385 else k,
               f"{kind} N={N} F={F} T={T}")


def test_every_point_flagged_over_full_chunks(xe, orc):
    """Two chunks of 32,768 samples and a rest: the counts of a chunk reach
    32,768 in 16-bit fields."""
    N, F, T, B = 33, 1, 2 * 32768 + 5, 32768
    flags = np.full((F, T, 2), 0xffffffff, np.uint32)
    _check(xe, orc, flags, None, N, B, 1, "all flagged")
