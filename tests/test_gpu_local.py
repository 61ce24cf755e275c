"""The local reduce (coarse bins) and the scan table's label search against the
CPU oracle: windows that hold the whole histogram and windows that move, steps
and runs with remainders, bins with more sessions than a run holds, stray and
unsorted times, byte counts up to 2^64 - 1, drops, accumulation, unaligned
columns, and narrow bins whose sessions are and are not in order enough."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _sessions(rng, n, span, jitter, order="sorted", big=False):
    t = (np.arange(n) + 0.5) * (span / n) + rng.uniform(-jitter, jitter, n)
    if order == "shuffled":
        t = rng.permutation(t)
    elif order == "stray":  # one session in 50 anywhere
        t = np.where(rng.random(n) < 0.02, rng.uniform(0, span, n), t)
    ts = np.clip(t, 0, span - 1).astype(np.uint32) + np.uint32(1000)
    by = np.exp(rng.normal(8, 2, n)).astype(np.uint64)
    if big:
        k = rng.integers(0, 64, n).astype(np.uint64)
        by = np.where(rng.random(n) < 0.3, (np.uint64(1) << k) - np.uint64(1), by)
        by[rng.random(n) < 0.01] = np.uint64(2**64 - 1)
    return ts, by


def _tables(sinet, kind):
    rng = np.random.default_rng(3)
    if kind == "edges":      # a scan table whose union starts at 0 and ends at the top
        base = np.array([0, 0x10000000, 0xFFFFFFFF, 0x80000000, 0x80000001], np.uint32)
        plen = np.array([8, 5, 32, 32, 32], np.uint8)
    elif kind == "all":
        base, plen = np.array([0, 0x0A000000], np.uint32), np.array([0, 8], np.uint8)
    elif kind == "scan":
        base, plen = rng.integers(0, 1 << 32, 64).astype(np.uint32), rng.integers(4, 25, 64).astype(np.uint8)
    else:
        base, plen = rng.integers(0, 1 << 32, 900).astype(np.uint32), rng.integers(6, 29, 900).astype(np.uint8)
    kw = {"kind": "trie", "inout_index": False} if kind == "trie" else {}
    return base, plen, sinet.Table(base, plen, **kw)


#        n, span, jitter, width, n_bins, order, big bytes, table
CASES = [
    (1, 1_000, 0, 1, 1, "sorted", False, "edges"),
    (1_025, 60_000, 3_000, 1_000, 60, "sorted", False, "edges"),
    (10_000, 60_000, 3_000, 1_000, 60, "sorted", True, "all"),
    (600_011, 60_000, 3_000, 86_400_000, 1, "sorted", True, "scan"),
    (700_001, 60_000, 3_000, 30, 2_000, "sorted", False, "nested"),
    (700_001, 60_000, 3_000, 29, 2_048, "sorted", False, "trie"),
    (900_003, 3_600_000, 5_000, 400, 9_000, "stray", True, "scan"),
    (900_003, 3_600_000, 5_000, 400, 8_000, "shuffled", False, "nested"),
    (1_500_007, 3_600_000, 5_000, 50, 72_000, "sorted", False, "trie"),
    (2_000_003, 600_000, 400, 7, 85_715, "sorted", True, "nested"),     # narrow bins, in order
    (2_000_003, 600_000, 90_000, 7, 85_715, "sorted", False, "scan"),   # narrow bins, not in order
]


@pytest.mark.parametrize("n,span,jitter,width,n_bins,order,big,kind", CASES)
def test_local_reduce_equals_oracle(n, span, jitter, width, n_bins, order, big, kind):
    import torch

    import paper_2106_12863_amd as sinet
    print("local", n, width, n_bins, order, kind, flush=True)
    rng = np.random.default_rng(n)
    base, plen, tab = _tables(sinet, kind)
    ts, by = _sessions(rng, n, span, jitter, order, big)
    edge = np.array([0, 1, 0x0FFFFFFF, 0x10000000, 0x17FFFFFF, 0x18000000, 0x80000000, 0x80000002,
                     0xFFFFFFFE, 0xFFFFFFFF], np.uint32)
    src, dst = (np.where(rng.random(n) < 0.2, rng.choice(edge, n),
                         rng.integers(0, 1 << 32, n).astype(np.uint32)) for _ in range(2))
    t0 = 900 if n_bins > 1 else 0  # the last bins' sessions are dropped where n_bins is short
    elab, ec, eb, ed = oracle.pipeline(base, plen, ts, src, dst, by, t0, width, n_bins)
    for off in (0, 1):
        def up(a, f):
            return f(np.concatenate([a[:off], a]))[off:]
        d = (up(ts, sinet.to_device_u32), up(src, sinet.to_device_u32), up(dst, sinet.to_device_u32),
             up(by, sinet.to_device_u64))
        want = bool(off) or kind != "trie"
        lab, out = sinet.pipeline(tab, *d, t0, width, n_bins, label=want)
        h = sinet.histogram(d[0], d[3], torch.from_numpy(elab).cuda(), t0, width, n_bins)
        sinet.histogram(d[0], d[3], torch.from_numpy(elab).cuda(), t0, width, n_bins, out=h,
                        accumulate=True)
        torch.cuda.synchronize()
        assert lab is None or np.array_equal(lab.cpu().numpy(), elab)
        for got, twice, e in zip(out, h, (ec, eb, ed)):
            assert np.array_equal(sinet.to_host_u64(got), e)
            assert np.array_equal(sinet.to_host_u64(twice), e + e)


@pytest.mark.parametrize("mode,n,n_bins,width", [
    ("window", 1_200_001, 9_000, 400),           # 130 sessions a bin: an event for every 16, in every piece
    ("window", 300_007, 2_100, 1),               # pieces that own few bins
    ("records", 3_000, 1, 1),                    # (always the local reduce)
    ("records", 200_003, 16_383 * 1_024, 1),     # one scan workgroup, and the first size past it
    ("records", 200_003, 16_384 * 1_024 - 1, 1),
    ("records", 5_000_011, 86_400, 50),          # runs of several chunks
])
def test_forced_reduces_equal_oracle(mode, n, n_bins, width):
    import torch

    import paper_2106_12863_amd as sinet
    print("forced", mode, n, n_bins, width, flush=True)
    rng = np.random.default_rng(n)
    span = n_bins * width
    ts, by = _sessions(rng, n, span, min(5_000, span / 3))
    lab = (rng.integers(0, 4, n) * (rng.random(n) < 0.3)).astype(np.uint8)
    exp = oracle.histogram(ts, by, lab, 1000, width, n_bins)
    d = sinet.to_device_u32(ts), sinet.to_device_u64(by), torch.from_numpy(lab).cuda()
    try:
        sinet.set_reduce(mode)
        out = sinet.histogram(*d, 1000, width, n_bins)
        sinet.histogram(*d, 1000, width, n_bins, out=out, accumulate=True)
        torch.cuda.synchronize()
    finally:
        sinet.set_reduce("auto")
    for got, e in zip(out, exp):
        assert np.array_equal(sinet.to_host_u64(got), e + e)


@pytest.mark.parametrize("chunk", [None, 2_048, 1 << 20])
def test_batch_with_coarse_streams_equals_oracle(chunk):
    """Streams of every reduce and label lookup in one plan, over two replays."""
    import torch

    import paper_2106_12863_amd as sinet
    cases = [CASES[0], CASES[2], (200_003, 60_000, 3_000, 1_000, 60, "sorted", True, "nested"),
             (300_001, 3_600_000, 5_000, 1_000, 3_000, "stray", True, "edges"),   # a moving window
             (150_001, 3_600_000, 5_000, 1_000, 3_000, "shuffled", False, "trie"),
             (100_003, 600_000, 5_000, 10, 60_000, "sorted", False, "nested"),    # records
             (120_007, 600_000, 5_000, 10, 60_000, "sorted", False, "trie")]
    streams, exps, keep = [], [], []
    for j, (n, span, jitter, width, n_bins, order, big, kind) in enumerate(cases):
        rng = np.random.default_rng(100 + j)
        base, plen, tab = _tables(sinet, kind)
        ts, by = _sessions(rng, n, span, jitter, order, big)
        src, dst = (rng.integers(0, 1 << 32, n).astype(np.uint32) for _ in range(2))
        exps.append(oracle.pipeline(base, plen, ts, src, dst, by, 900, width, n_bins))
        lab = torch.empty(n, dtype=torch.uint8, device="cuda") if j % 2 == 0 else None
        out = [torch.full_like(t, -1) for t in sinet.new_hist(n_bins)]
        keep.append((lab, out))
        streams.append(sinet.BatchStream(tab, sinet.to_device_u32(ts), sinet.to_device_u32(src),
                                         sinet.to_device_u32(dst), sinet.to_device_u64(by), 900, width,
                                         n_bins, label=lab, out=out))
    print("batch of coarse streams", chunk, flush=True)
    tune = None
    if chunk:
        tune = sinet.Tune()
        tune.block, tune.chunk, tune.grid = 512, chunk, 0
    plan = sinet.BatchPlan(streams, tune)
    for _ in range(2):
        plan.run()
        torch.cuda.synchronize()
        for j, ((lab, out), (elab, ec, eb, ed)) in enumerate(zip(keep, exps)):
            assert lab is None or np.array_equal(lab.cpu().numpy(), elab), j
            for got, e in zip(out, (ec, eb, ed)):
                assert np.array_equal(sinet.to_host_u64(got), e), j


def test_labels_in_pieces():
    """More sessions than the workspace holds labels of, by a table whose lookups
    are a pass of their own: equal to the histogram of the labels given."""
    import torch

    import paper_2106_12863_amd as sinet
    n, width, n_bins = (1 << 28) + 4_099, 60_000, 1_440
    rng = np.random.default_rng(5)
    base, plen = rng.integers(0, 1 << 32, 900).astype(np.uint32), rng.integers(6, 29, 900).astype(np.uint8)
    tab = sinet.Table(base, plen, kind="trie", inout_index=False)
    print("labels in pieces", n, flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(6)
    ts = torch.linspace(0, n_bins * width - 1, n, device="cuda", dtype=torch.float64).to(torch.int32)
    src, dst = (torch.randint(-(1 << 31), 1 << 31, (n,), generator=g, device="cuda", dtype=torch.int32)
                for _ in range(2))
    by = torch.randint(0, 1 << 31, (n,), generator=g, device="cuda")
    lab = sinet.discriminate(tab, src, dst)[0]
    given = sinet.histogram(ts, by, lab, 60_000, width, n_bins)
    none, looked = sinet.pipeline(tab, ts, src, dst, by, 60_000, width, n_bins, label=False)
    torch.cuda.synchronize()
    assert none is None and int(given[0].sum()) + int(given[2][:, 0].sum()) == n
    for a, b in zip(given, looked):
        assert torch.equal(a, b)
    sinet.pipeline(tab, ts, src, dst, by, 60_000, width, n_bins, label=False, out=looked, accumulate=True)
    torch.cuda.synchronize()
    for a, b in zip(given, looked):
        assert torch.equal(a * 2, b)
