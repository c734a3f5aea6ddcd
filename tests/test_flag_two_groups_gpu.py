"""Flag counts of two 128-input groups on either side of the line between the
two Gram kernels, at 512 units of tiles (GPU); the wide kernel then has no pairs
of super blocks.  Counts must equal the oracle's, added to what the array held.
"""

import numpy as np
import pytest

import oracle
from paper_1503_06189_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("N,F", [(129, 128), (129, 129), (224, 129), (225, 129), (256, 128),
                                 (256, 129)])
def test_two_groups(N, F):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1503_06189_amd import xengine as xe
    rng = np.random.default_rng(900 + N + F)
    for T, offset, run in ((33, 0, 1), (150, 1, 32), (2100, 0, 32)):
        print(f"flags N={N} F={F} T={T} offset={offset}", flush=True)
        B = 16
        flags = (synth.fengine_flags(rng, T, F, N, 0.01, mean_run=32.0, garbage_padding=True)
                 if run > 1 else synth.random_flags(rng, T, F, N, 0.03, garbage_padding=True))
        mask = synth.bernoulli_mask(rng, F, T, B, 0.1)
        _, want = oracle.load().flag_counters(flags, mask, N, B)
        buf = torch.empty(flags.size + offset, dtype=torch.int32, device="cuda")
        buf[offset:] = torch.from_numpy(np.ascontiguousarray(flags).view(np.int32).ravel()).cuda()
        d = xe.new_flag_counts(N, F)
        d += 3
        xe.flag_accumulate(buf[offset:].view(flags.shape), torch.from_numpy(mask).cuda(), B, N, d)
        assert np.array_equal(d.cpu().numpy().astype(np.int64), want + 3)
