"""Plans of the widest frames that the ABI accepts (F * N up to XE_MAX_FN).

Above F * N = 3,355,443 the offset bound leaves no steps for a chunk beside its
lookahead; such frames run in the shortest chunks.  The queries run in a
process of their own, because a plan without steps divides by zero.
"""

import json
import os
import subprocess
import sys

import pytest

from paper_1503_06189_amd import xengine as xe

WIDEST = 4194304
LAST_LONG = 3355443        # the last F * N whose bound leaves 4 steps

CHILD = """
import ctypes, json, sys
from paper_1503_06189_amd import xengine as xe
N, F, T = map(int, sys.argv[1:])
def attempt(call):
    try:
        return call()
    except xe.XEngineError as e:
        return e.status
p = attempt(lambda: xe.plan_query(N, F, T, 256, 256))
b = attempt(lambda: xe.batch_query([(N, F, T, 256)], n_cu=256))
s = xe.lib().xe_accumulate_noalloc(ctypes.c_void_p(0x1000), None, N, F, T, 256,
                                   ctypes.c_void_p(0x2000), ctypes.c_void_p(0x3000), None) \\
    if T > 128 else None
print(json.dumps([p if isinstance(p, int) else [p.splits, p.steps_per_split],
                  b if isinstance(b, int) else [b.items, b.unaligned], s]))
"""


def _query(N, F, T):
    r = subprocess.run([sys.executable, "-c", CHILD, str(N), str(F), str(T)],
                       capture_output=True, text=True, timeout=120, cwd=os.path.dirname(xe.HERE))
    assert r.returncode == 0, (r.returncode, r.stderr[-500:])
    return json.loads(r.stdout.strip().splitlines()[-1])


@pytest.mark.parametrize("N,F,batch", [
    (1, WIDEST, [0, 1]), (1, LAST_LONG, [0, 1]), (1, LAST_LONG + 1, [0, 1]),
    (127, 33026, [0, 1]), (128, 32768, [32768, 0]), (256, 16384, [16384, 0]),
    (4096, 1024, xe.XE_ERR_WORKSPACE),     # more items than a work list holds
])
def test_short_frames_run_in_one_chunk(N, F, batch):
    assert LAST_LONG <= N * F <= WIDEST
    for T in (1, 32, 128):
        assert _query(N, F, T)[:2] == [[1, 4], batch]


@pytest.mark.parametrize("N,F", [(1, WIDEST), (128, 32768), (4096, 1024)])
def test_longer_frames_do_not_fit_the_workspace(N, F):
    # (chunks of 4 steps: the second one's sums are larger than any workspace
    # that the queries assume)
    plan, _, noalloc = _query(N, F, 129)
    assert plan == xe.XE_ERR_WORKSPACE and noalloc == xe.XE_ERR_WORKSPACE


@pytest.mark.parametrize("N,F,T,want", [(256, 64, 16384, [4, 128]), (2048, 16, 8192, [1, 256]),
                                        (256, 2048, 4096, [2, 108]), (128, 20480, 96, [1, 4])])
def test_chunks_of_narrower_frames_are_unchanged(N, F, T, want):
    assert _query(N, F, T)[0] == want
