"""Performance cases of the correlator: the work a user's program has it do.

Each case is one pass through the public entry points of
``paper_1503_06189_amd.xengine``, on device-resident inputs made from a
seed.  Integrations start from an overwriting call or cleared sums in every
pass, so a pass can be repeated on the same state and always returns the
same values.

Kinds and what they stand for:

integrate  a short integration and its normalisation: the first frame
           overwrites the sums, the others extend them, then V / n
serve      what a streaming server enqueues for one frame of each of its
           streams: the frame's time slices, one batch per slice index
batch      uneven single-channel instances run as one planned batch
flags      per-baseline intersections of one frame's per-input flags
assemble   one frame built from the F-engine's packets
shift      per-input delays applied to a frame and its flags
pipeline   packets to normalised visibilities, every stage in order
"""

import math
import random

import torch

from paper_1503_06189_amd import xengine

DEV = "cuda"
#: samples drawn at a time; bounds the scratch memory of the generators
CHUNK_BYTES = 1 << 25


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------

def listed():
    return [
        # the smallest call: a bench-top array of 16 inputs, launch latency counts
        dict(name="tiny_n16", kind="integrate", N=16, F=8, T=256, B=256, frames=1, loss=0.0),
        # one stream of a server: 128 inputs, 4096-sample frames
        dict(name="stream_n128", kind="integrate", N=128, F=40, T=4096, B=256, frames=2,
             loss=0.02),
        # one server's share of the 256-input array, 256 MiB frames
        dict(name="pathfinder", kind="integrate", N=256, F=64, T=16384, B=256, frames=2,
             loss=0.01),
        # the full array: 2048 inputs, 16 channels on one GPU
        dict(name="large_n2048", kind="integrate", N=2048, F=16, T=8192, B=256, frames=1,
             loss=0.005),
        # an array with dead inputs cut out: no size is a multiple of anything
        dict(name="ragged_n250", kind="integrate", N=250, F=33, T=5001, B=100, frames=2,
             loss=0.03),
        # 8 streams sharing a GPU, 4096-sample frames copied in 1024-sample slices
        dict(name="serve_8_streams", kind="serve", streams=8, T=4096, slices=4, B=256,
             shapes=105, loss=0.02),
        # 128 sub-array instances of very different sizes in one planned batch
        dict(name="batch_128_uneven", kind="batch", n_inst=128, shapes=104, t_max=65536,
             n_max=1024, odd=False, loss=0.02),
        # the F-engine's usual flags: rare bursts on single inputs
        dict(name="flags_bursty_n256", kind="flags", N=256, F=64, T=16384, B=256, rate=0.001,
             run=32.0, loss=0.01),
        # a noisy site: 5% of all points flagged independently, 512 inputs
        dict(name="flags_scattered_n512", kind="flags", N=512, F=32, T=8192, B=256, rate=0.05,
             run=1.0, loss=0.01),
        # one server's 8 links, 1% of the packets dropped, some twice or late
        dict(name="assemble_pathfinder", kind="assemble", N=256, S=8, T=16384, drop=0.01,
             dup=0.005, rate=0.001),
        # cable delays of a few samples
        dict(name="shift_pathfinder", kind="shift", N=256, F=64, T=16384, delay=8, rate=0.001),
        # a frame's whole way through the GPU
        dict(name="pipeline_pathfinder", kind="pipeline", N=256, S=8, T=16384, drop=0.01,
             dup=0.005, rate=0.001),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _inputs(rng, lo, hi):
    """A number of inputs: round ones half of the time, any otherwise."""
    n = _log(rng, lo, hi)
    return max(lo, min(hi, 16 * round(n / 16))) if rng.random() < 0.5 else n


def draw(rng):
    kind = rng.choice(["integrate"] * 5 + ["serve", "batch", "flags", "flags", "assemble",
                                           "shift", "shift", "pipeline"])
    loss = rng.choice([0.0, round(rng.uniform(0.001, 0.08), 4)])
    if kind == "integrate":
        N, F, T = _inputs(rng, 8, 2048), _log(rng, 1, 128), _log(rng, 128, 16384)
        frames = rng.choice([1, 2])
        most = 8 * (2048 * 2049 // 2) * 16 * 8192
        while 8 * (N * (N + 1) // 2) * F * T * frames > most or N * F * T * frames > 1 << 29:
            F, T = max(1, F // 2), max(128, T * 3 // 4)
        return dict(kind=kind, N=N, F=F, T=T, B=rng.choice([4, 64, 100, 256, _log(rng, 16, 2048)]),
                    frames=frames, loss=loss)
    if kind == "serve":
        slices = rng.choice([1, 2, 4, 8])
        B = rng.choice([64, 128, 256])
        return dict(kind=kind, streams=rng.randint(1, 8), T=slices * B * rng.randint(1, 2048 // B),
                    slices=slices, B=B, shapes=rng.randrange(1 << 16), loss=loss)
    if kind == "batch":
        return dict(kind=kind, n_inst=_log(rng, 4, 128), shapes=rng.randrange(1 << 16),
                    t_max=_log(rng, 2048, 65536), n_max=rng.choice([128, 256, 512, 1024]),
                    odd=rng.random() < 0.3, loss=loss)
    N = _inputs(rng, 16, 1024)
    rate = round(math.exp(rng.uniform(math.log(1e-4), math.log(0.05))), 6)
    if kind == "flags":
        F, T = _log(rng, 1, 64), _log(rng, 200, 16384)
        while N * F * T > 256 * 64 * 16384:
            F, T = max(1, F // 2), max(200, T * 3 // 4)
        run = rng.choice([1.0, 32.0])
        if rng.random() < 0.1:
            rate, run = 0.5, 1.0     # a broken site
        return dict(kind=kind, N=N, F=F, T=T, B=rng.choice([4, 100, 256]), rate=rate, run=run,
                    loss=loss)
    if kind == "shift":
        F, T = _log(rng, 1, 64), _log(rng, 200, 16384)
        while N * F * T > 256 * 64 * 16384:
            F, T = max(1, F // 2), max(200, T * 3 // 4)
        return dict(kind=kind, N=N, F=F, T=T, delay=_log(rng, 1, 100), rate=rate)
    S, T = rng.randint(1, 8), 4 * _log(rng, 64, 4096)
    while N * 8 * S * T > 256 * 64 * 16384:
        S, T = max(1, S // 2), max(256, 4 * (T // 6))
    return dict(kind=kind, N=N, S=S, T=T, drop=rng.choice([0.0, 0.01, 0.1]),
                dup=rng.choice([0.0, 0.005]), rate=rate)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) % (1 << 62))
    return g


def _quantise(re, im):
    re = re.round_().clamp_(-7, 7).add_(8).to(torch.uint8)
    im = im.round_().clamp_(-7, 7).add_(8).to(torch.uint8)
    return (re << 4) | im


def _voltages(g, T, F, N, sigma=2.5, amp=2.0):
    """uint8 [T, F, N]: receiver noise plus one sky tone per channel, seen by
    each input through its own complex gain; 4+4-bit offset-encoded."""
    r = torch.rand(N, generator=g, device=DEV) + 0.5
    theta = torch.rand(N, generator=g, device=DEV) * (2 * math.pi)
    nu = torch.rand(F, generator=g, device=DEV) - 0.5
    phi = torch.rand(F, generator=g, device=DEV) * (2 * math.pi)
    out = torch.empty((T, F, N), dtype=torch.uint8, device=DEV)
    step = max(1, CHUNK_BYTES // (F * N))
    for t0 in range(0, T, step):
        t1 = min(T, t0 + step)
        t = torch.arange(t0, t1, device=DEV, dtype=torch.float64)[:, None]
        arg = ((t * nu.double()) % 1.0).float() * (2 * math.pi) + phi
        arg = arg[:, :, None] + theta
        re = torch.randn((t1 - t0, F, N), generator=g, device=DEV).mul_(sigma)
        im = torch.randn((t1 - t0, F, N), generator=g, device=DEV).mul_(sigma)
        re.addcmul_(torch.cos(arg), r, value=amp)
        im.addcmul_(torch.sin(arg), r, value=amp)
        out[t0:t1] = _quantise(re, im)
    return out


def _noise(g, n, sigma=2.5):
    """uint8 [n]: quantised noise without a layout."""
    out = torch.empty(n, dtype=torch.uint8, device=DEV)
    for k in range(0, n, CHUNK_BYTES):
        m = min(CHUNK_BYTES, n - k)
        out[k:k + m] = _quantise(torch.randn(m, generator=g, device=DEV).mul_(sigma),
                                 torch.randn(m, generator=g, device=DEV).mul_(sigma))
    return out


def _loss_mask(g, F, T, B, p):
    return (torch.rand((F, -(-T // B)), generator=g, device=DEV) < p).to(torch.uint8)


def _valid(mask, T, B):
    """bool [T, F] of the samples outside lost blocks."""
    return (mask == 0).repeat_interleave(B, dim=1)[:, :T].t()


def _zero_lost(packed, mask, B):
    """The network thread's zero fill."""
    if bool(mask.any()):
        packed.masked_fill_(~_valid(mask, packed.shape[0], B)[:, :, None], 0x88)
    return packed


def _flag_words(g, F, T, N, rate, run):
    """int32 [F, T, ceil(N/32)] bit-fields: runs of flagged samples of mean
    length ``run`` on single inputs, ``rate`` of all points in total."""
    W = -(-N // 32)
    if run <= 1.0 and rate >= 0.02:          # independent points
        out = torch.empty((F, T, W), dtype=torch.int32, device=DEV)
        weight = (torch.ones(32, dtype=torch.int64, device=DEV)
                  << torch.arange(32, device=DEV)).to(torch.int64)
        keep = (torch.arange(W * 32, device=DEV) < N).view(W, 32)
        step = max(1, CHUNK_BYTES // (T * W * 32))
        for f0 in range(0, F, step):
            f1 = min(F, f0 + step)
            bits = torch.rand((f1 - f0, T, W, 32), generator=g, device=DEV) < rate
            words = ((bits & keep) * weight).sum(dim=-1)
            out[f0:f1] = torch.where(words >= 1 << 31, words - (1 << 32), words).to(torch.int32)
        return out
    n = max(1, int(F * N * T * rate / run))
    f = torch.randint(0, F, (n,), generator=g, device=DEV)
    i = torch.randint(0, N, (n,), generator=g, device=DEV)
    t = torch.randint(0, T, (n,), generator=g, device=DEV)
    u = torch.rand(n, generator=g, device=DEV).clamp_(1e-7, 1.0)
    length = (u.log() / math.log(1.0 - 1.0 / run)).long() + 1 if run > 1.0 else torch.ones_like(f)
    first = torch.cumsum(length, 0) - length
    at = torch.arange(int(length.sum()), device=DEV)
    own = torch.repeat_interleave(torch.arange(n, device=DEV), length)
    tt = t[own] + at - first[own]
    ok = tt < T
    point = torch.unique(((f[own] * T + tt) * N + i[own])[ok])
    ii = point % N
    words = torch.zeros(F * T * W, dtype=torch.int64, device=DEV)
    words.index_add_(0, (point // N) * W + ii // 32, torch.ones_like(ii) << (ii % 32))
    words = torch.where(words >= 1 << 31, words - (1 << 32), words)
    return words.to(torch.int32).view(F, T, W)


def _flag_bits(words, f, N):
    """bool [T, N] of channel f."""
    w = words[f].long() & 0xffffffff
    bits = (w[:, :, None] >> torch.arange(32, device=words.device)) & 1
    return bits.reshape(w.shape[0], -1)[:, :N].bool()


def _observation(case, seed):
    """A frame, its flags, and which packets of it were dropped."""
    g = _gen(seed)
    F = 8 * case["S"]
    packed = _voltages(g, case["T"], F, case["N"])
    flags = _flag_words(g, F, case["T"], case["N"], case["rate"], 32.0)
    dropped = torch.rand((case["T"] // 4, case["S"]), generator=g, device=DEV) < case["drop"]
    return g, packed, flags, dropped


def _packets(case, g, packed, flags, dropped):
    """uint8 [n, packet_bytes]: the frame as the F-engine's packets, in
    arrival order: dropped ones missing, some twice (the copy later and with
    another payload), reordered within 64 packets."""
    T, F, N = packed.shape
    S, K, W = F // 8, T // 4, -(-N // 32)
    n, pb = K * S, xengine.packet_bytes(N)
    out = torch.empty((n, pb), dtype=torch.uint8, device=DEV)
    out[:, 16:16 + 32 * N] = packed.view(K, 4, S, 8, N).permute(0, 2, 1, 3, 4).reshape(n, 32 * N)
    words = flags.view(S, 8, K, 4, W).permute(2, 0, 3, 1, 4).reshape(n, 32 * W).contiguous()
    out[:, 16 + 32 * N:] = words.view(torch.uint8)
    head = torch.empty((n, 2), dtype=torch.int64, device=DEV)
    head[:, 0] = torch.arange(n, device=DEV) // S
    head[:, 1] = (torch.arange(n, device=DEV) % S) + (N << 32)
    out[:, :16] = head.view(torch.uint8)
    kept = (~dropped).reshape(-1).nonzero().flatten()
    twice = kept[torch.rand(kept.numel(), generator=g, device=DEV) < case["dup"]]
    at = torch.cat([kept + torch.rand(kept.numel(), generator=g, device=DEV) * 64,
                    twice + 64 + torch.rand(twice.numel(), generator=g, device=DEV) * 64])
    order = torch.argsort(at)
    rows = torch.cat([kept, twice])[order]
    copy = torch.cat([torch.zeros_like(kept), torch.ones_like(twice)])[order].bool()
    sent = out[rows]
    where = copy.nonzero().flatten()
    if where.numel():
        sent[where, 16:] = torch.randint(0, 256, (where.numel(), pb - 16), generator=g,
                                         device=DEV, dtype=torch.uint8)
    return sent


def _stream_shapes(case):
    rng = random.Random(case["shapes"])
    return [(rng.choice([128, 256, 512]), rng.randint(16, 64)) for _ in range(case["streams"])]


def _batch_shapes(case):
    rng = random.Random(case["shapes"])
    out = []
    for _ in range(case["n_inst"]):
        if case["odd"]:
            N = _log(rng, 17, case["n_max"])
        else:
            N = rng.choice([n for n in (64, 128, 256, 512, 1024) if n <= case["n_max"]])
        T = _log(rng, 1024, case["t_max"])
        out.append((N, T if case["odd"] else max(256, 256 * round(T / 256))))
    return out


class _Sums:
    """Sums and counts of several integrations in two flat buffers."""

    def __init__(self, shapes):
        pairs = [F * (N * (N + 1) // 2) for N, F in shapes]
        self.vis = torch.zeros((sum(pairs), 2), dtype=torch.int32, device=DEV)
        self.count = torch.zeros(sum(F for _, F in shapes), dtype=torch.int64, device=DEV)
        self.each, p, c = [], 0, 0
        for (N, F), n in zip(shapes, pairs):
            self.each.append((self.vis[p:p + n].view(F, N * (N + 1) // 2, 2),
                              self.count[c:c + F]))
            p, c = p + n, c + F

    def clear(self):
        self.vis.zero_()
        self.count.zero_()
        for v, _ in self.each:
            xengine.reset_integration(v)


def _flat_frames(g, shapes):
    """Noise frames [T, F, N] of the shapes, 256-byte aligned in one buffer."""
    at, n = [], 0
    for T, F, N in shapes:
        at.append(n)
        n += -(-T * F * N // 256) * 256
    flat = _noise(g, n)
    return [flat[a:a + T * F * N].view(T, F, N) for a, (T, F, N) in zip(at, shapes)]


def prepare(case, seed):
    kind = case["kind"]
    s = dict(case=case)
    if kind == "integrate":
        g = _gen(seed)
        N, F, T, B = case["N"], case["F"], case["T"], case["B"]
        s["frames"] = []
        for _ in range(case["frames"]):
            packed = _voltages(g, T, F, N)
            mask = _loss_mask(g, F, T, B, case["loss"])
            s["frames"].append((_zero_lost(packed, mask, B), mask))
        s["vis"], s["count"] = xengine.new_accumulators(N, F, torch.device(DEV))
        s["out"] = torch.empty(s["vis"].shape, dtype=torch.float32, device=DEV)
    elif kind == "serve":
        g = _gen(seed)
        shapes = _stream_shapes(case)
        s["sums"] = _Sums(shapes)
        frames = _flat_frames(g, [(case["T"], F, N) for N, F in shapes])
        n, B = case["T"] // case["slices"], case["B"]
        s["batches"] = [[] for _ in range(case["slices"])]
        for packed, (vis, count) in zip(frames, s["sums"].each):
            mask = _loss_mask(g, packed.shape[1], case["T"], B, case["loss"])
            _zero_lost(packed, mask, B)
            for k in range(case["slices"]):
                part = mask[:, k * n // B:(k + 1) * n // B].contiguous()
                s["batches"][k].append((packed[k * n:(k + 1) * n], part, B, vis, count))
    elif kind == "batch":
        g = _gen(seed)
        shapes = _batch_shapes(case)
        s["sums"] = _Sums([(N, 1) for N, _ in shapes])
        frames = _flat_frames(g, [(T, 1, N) for N, T in shapes])
        items = []
        for packed, (vis, count) in zip(frames, s["sums"].each):
            mask = _loss_mask(g, 1, packed.shape[0], 256, case["loss"])
            items.append((_zero_lost(packed, mask, 256), mask, 256, vis, count))
        s["plan"] = xengine.BatchPlan(items)
    elif kind == "flags":
        g = _gen(seed)
        s["flags"] = _flag_words(g, case["F"], case["T"], case["N"], case["rate"], case["run"])
        s["mask"] = _loss_mask(g, case["F"], case["T"], case["B"], case["loss"])
        s["dcount"] = xengine.new_flag_counts(case["N"], case["F"], torch.device(DEV))
    elif kind == "shift":
        g = _gen(seed)
        s["packed"] = _voltages(g, case["T"], case["F"], case["N"])
        s["flags"] = _flag_words(g, case["F"], case["T"], case["N"], case["rate"], 32.0)
        s["delays"] = torch.randint(-case["delay"], case["delay"] + 1, (case["N"],), generator=g,
                                    device=DEV, dtype=torch.int32)
        s["out"], s["flags_out"] = torch.empty_like(s["packed"]), torch.empty_like(s["flags"])
    else:
        g, packed, flags, dropped = _observation(case, seed)
        s["packets"] = _packets(case, g, packed, flags, dropped)
        T, F, N = packed.shape
        s["frame"] = (packed, torch.empty((F, T // 4), dtype=torch.uint8, device=DEV), flags,
                      torch.empty(6, dtype=torch.int64, device=DEV))
        packed.zero_()      # the frame's buffers are reused for what is assembled
        flags.zero_()
        if kind == "pipeline":
            s["vis"], s["count"] = xengine.new_accumulators(N, F, torch.device(DEV))
            s["dcount"] = xengine.new_flag_counts(N, F, torch.device(DEV))
            s["out"] = torch.empty(s["vis"].shape, dtype=torch.float32, device=DEV)
            s["n"] = torch.empty(s["dcount"].shape, dtype=torch.int32, device=DEV)
    return s


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "integrate":
        vis, count = state["vis"], state["count"]
        for k, (packed, mask) in enumerate(state["frames"]):
            if k == 0:
                xengine.correlate_frame(packed, mask, case["B"], vis, count)
            else:
                xengine.accumulate(packed, mask, case["B"], vis, count)
        out = xengine.normalize(vis, count, state["out"])
        return dict(vis=vis, count=count, out=out)
    if kind == "serve":
        state["sums"].clear()
        for items in state["batches"]:
            xengine.accumulate_batch(items)
        return dict(vis=state["sums"].vis, count=state["sums"].count)
    if kind == "batch":
        state["sums"].clear()
        state["plan"].run()
        return dict(vis=state["sums"].vis, count=state["sums"].count)
    if kind == "flags":
        state["dcount"].zero_()
        return xengine.flag_accumulate(state["flags"], state["mask"], case["B"], case["N"],
                                       state["dcount"])
    if kind == "shift":
        return xengine.time_shift(state["packed"], state["delays"], state["flags"], state["out"],
                                  state["flags_out"])
    packed, mask, flags, stats = xengine.assemble_frame(
        state["packets"], case["N"], case["S"], 0, 0, case["T"], *state["frame"])
    if kind == "assemble":
        return dict(packed=packed, mask=mask, flags=flags, stats=stats)
    xengine.apply_flags(packed, flags)
    vis, count = xengine.correlate_frame(packed, mask, 4, state["vis"], state["count"])
    state["dcount"].zero_()
    xengine.flag_accumulate(flags, mask, 4, case["N"], state["dcount"])
    out = xengine.normalize_flagged(vis, count, state["dcount"], state["out"], state["n"])
    return dict(vis=vis, count=count, dcount=state["dcount"], out=out, n=state["n"])


def _correlation(N, F, T):
    P = N * (N + 1) // 2
    return 8 * P * F * T, N * F * T, 8 * P * F


def work(case):
    kind = case["kind"]
    if kind == "integrate":
        ops, frame, sums = _correlation(case["N"], case["F"], case["T"])
        k = case["frames"]
        return dict(bytes=k * frame + 2 * sums, flops=k * ops)
    if kind in ("serve", "batch"):
        if kind == "serve":
            parts = [_correlation(N, F, case["T"]) for N, F in _stream_shapes(case)]
        else:
            parts = [_correlation(N, 1, T) for N, T in _batch_shapes(case)]
        return dict(bytes=sum(p[1] + p[2] for p in parts), flops=sum(p[0] for p in parts))
    N, T = case["N"], case["T"]
    F = case["F"] if "F" in case else 8 * case["S"]
    P, W = N * (N + 1) // 2, -(-N // 32)
    words = 4 * F * T * W
    if kind == "flags":
        return dict(bytes=words + 4 * P * F, flops=0)
    if kind == "shift":
        return dict(bytes=2 * (N * F * T + words), flops=0)
    n = int(F // 8 * (T // 4) * (1 - case["drop"]) * (1 + case["dup"]))
    packets = n * xengine.packet_bytes(N)
    if kind == "assemble":
        return dict(bytes=packets + N * F * T + words + F * T // 4, flops=0)
    # sums, normalised values, intersections and sample counts come back
    return dict(bytes=packets + F * P * (8 + 8 + 4 + 4), flops=8 * P * F * T)


# ---------------------------------------------------------------------------
# the same values in 64 bits
# ---------------------------------------------------------------------------

def _products(byte, keep):
    """Re, Im of V (float64 [N, N]) of one channel's bytes [T, N], points
    outside ``keep`` counted as 0."""
    a = ((byte >> 4).double() - 8) * keep
    b = ((byte & 15).double() - 8) * keep
    at, bt = a.t().contiguous(), b.t().contiguous()
    return at @ a + bt @ b, bt @ a - at @ b


def exact(case, seed):
    kind = case["kind"]
    if kind not in ("integrate", "pipeline"):
        return None          # integers and bytes only
    N, T = case["N"], case["T"]
    F = case["F"] if "F" in case else 8 * case["S"]
    i, j = torch.triu_indices(N, N, device=DEV)
    out = torch.zeros((F, N * (N + 1) // 2, 2), dtype=torch.float64, device=DEV)
    if kind == "integrate":
        g = _gen(seed)
        n = torch.zeros(F, dtype=torch.float64, device=DEV)
        for _ in range(case["frames"]):
            packed = _voltages(g, T, F, N)
            mask = _loss_mask(g, F, T, case["B"], case["loss"])
            valid = _valid(mask, T, case["B"]).double()
            n += valid.sum(dim=0)
            for f in range(F):
                re, im = _products(packed[:, f, :], valid[:, f, None])
                out[f, :, 0] += re[i, j]
                out[f, :, 1] += im[i, j]
        out = torch.where(n[:, None, None] > 0, out / n[:, None, None].clamp(min=1), 0.0)
        return dict(vis=None, count=None, out=out)
    _, packed, flags, dropped = _observation(case, seed)
    there = (~dropped).repeat_interleave(4, dim=0)          # [T, S]
    for f in range(F):
        keep = (there[:, f // 8, None] & ~_flag_bits(flags, f, N)).double()
        re, im = _products(packed[:, f, :], keep)
        n = (keep.t().contiguous() @ keep)[i, j]
        out[f, :, 0] = torch.where(n > 0, re[i, j] / n.clamp(min=1), 0.0)
        out[f, :, 1] = torch.where(n > 0, im[i, j] / n.clamp(min=1), 0.0)
    return dict(vis=None, count=None, dcount=None, out=out, n=None)
