"""Per-baseline normalisation at the edges of its row pairs (GPU).

Frames of up to 128 inputs take one thread per baseline, larger ones rows i and
N - 1 - i together.  The quotients are formed from a
shared reciprocal and must equal double division rounded once to float, bit for
bit, on extreme sums and counts too.
"""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def xe():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1503_06189_amd import xengine
    xengine.lib()   # fails loudly if the library is missing
    return xengine


@pytest.mark.parametrize("N", [1, 2, 3, 64, 127, 128, 129, 130, 254, 255, 256, 257, 511, 512, 600,
                               2049])
def test_quotients_equal_double_division(xe, N):
    rng = np.random.default_rng(60 + N)
    F = 3 if N < 1000 else 1
    P = N * (N + 1) // 2
    i, j = np.triu_indices(N)
    vis = rng.integers(-2 ** 31, 2 ** 31, (F, P, 2), dtype=np.int64)
    vis[:, ::3] = rng.integers(-1000, 1000, vis[:, ::3].shape)
    count = rng.integers(1, 2 ** 40, F)
    count[0] = 5
    d = rng.integers(0, 4, (F, P))
    if F > 1:
        d[1] = rng.integers(0, 2 ** 31 - 1, P)
    diag = np.flatnonzero(i == j)
    n = count[:, None] - d[:, diag][:, i] - d[:, diag][:, j] + d
    with np.errstate(divide="ignore", invalid="ignore"):
        want = np.where(n[..., None] == 0, 0.0, vis.astype(np.float64) / n[..., None].astype(np.float64))
    print(f"normalize N={N} F={F}", flush=True)
    dev = lambda x, t: torch.from_numpy(x.astype(t)).cuda()
    n_out = torch.empty((F, P), dtype=torch.int32, device="cuda")
    out = xe.normalize_flagged(dev(vis, np.int32), dev(count, np.int64), dev(d, np.int32),
                               n_out=n_out)
    out = out[0] if isinstance(out, tuple) else out
    got = out.cpu().numpy().reshape(F, P, -1)
    if got.dtype == np.complex64:
        got = np.stack([got.real, got.imag], axis=-1).reshape(F, P, 2)
    assert np.array_equal(got.view(np.uint32), want.astype(np.float32).view(np.uint32))
    assert np.array_equal(n_out.cpu().numpy(), n.astype(np.int32))
