"""Coarse streams of a batch whose tables walk global memory (no in/out index):
their labels come from the lookup pass, whole and moving windows, against the CPU
oracle and the labels; and streams whose sessions are out of order."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _stream(sinet, torch, tab, base, plen, seed, n, width, n_bins, order, label):
    rng = np.random.default_rng(seed)
    t = (np.arange(n) + 0.5) * (n_bins * width / n) + rng.uniform(-4_000, 4_000, n)
    if order == "shuffled":
        t = rng.permutation(t)
    elif order == "half":
        t[n // 2:] = rng.permutation(t[n // 2:])
    ts = (np.clip(t, 0, n_bins * width + 700) + 300).astype(np.uint32)
    by = (np.uint64(1) << rng.integers(0, 60, n).astype(np.uint64)) + rng.integers(0, 9, n).astype(np.uint64)
    ends = np.where(rng.random((2, n)) < 0.5, rng.integers(0, 1 << 32, (2, n)),
                    base[rng.integers(0, len(base), (2, n))] + rng.integers(-2, 300, (2, n))) & 0xFFFFFFFF
    src, dst = ends.astype(np.uint32)
    exp = oracle.pipeline(base, plen, ts, src, dst, by, 300, width, n_bins)
    lab = torch.full((n,), 9, dtype=torch.uint8, device="cuda") if label else None
    out = [torch.full_like(x, -1) for x in sinet.new_hist(n_bins)]
    s = sinet.BatchStream(tab, sinet.to_device_u32(ts), sinet.to_device_u32(src), sinet.to_device_u32(dst),
                          sinet.to_device_u64(by), 300, width, n_bins, label=lab, out=out)
    return s, lab, out, exp


def _check(sinet, torch, plan, made):
    for _ in range(3):
        plan.run()
        torch.cuda.synchronize()
        for j, (_, lab, out, (elab, *exp)) in enumerate(made):
            assert lab is None or np.array_equal(lab.cpu().numpy(), elab), j
            for got, e in zip(out, exp):
                assert np.array_equal(sinet.to_host_u64(got), e), j


@pytest.mark.parametrize("kind", ["trie", "pla", "pla_wide", "mlp", "bsearch"])
def test_coarse_streams_of_searching_tables_equal_oracle(kind):
    import torch

    import paper_2106_12863_amd as sinet
    rng = np.random.default_rng(6)
    base = (rng.integers(0, 1 << 32, 30_000) & ~0xFF).astype(np.uint32)
    plen = rng.integers(14, 30, 30_000).astype(np.uint8)
    tab = sinet.Table(base, plen, kind=kind.split("_")[0], inout_index=False)
    if kind == "pla_wide":
        tab.train(segments=200)
    elif kind in ("pla", "mlp"):
        tab.train(steps=50 if kind == "mlp" else 0)
    cuts = [(150_001, 60_000, 60, True), (150_003, 60_000, 60, False),          # whole
            (400_009, 1_000, 3_000, True), (400_011, 1_000, 3_000, False),      # a moving window
            (90_001, 10, 40_000, True), (5, 1_000, 3, False)]                   # records; a few
    print("batch lookups", kind, flush=True)
    made = [_stream(sinet, torch, tab, base, plen, j, n, w, b, "sorted", lab)
            for j, (n, w, b, lab) in enumerate(cuts)]
    _check(sinet, torch, sinet.BatchPlan([m[0] for m in made]), made)


@pytest.mark.parametrize("order,records", [("shuffled", False), ("half", True), ("sorted", True)])
def test_coarse_streams_set_aside_equal_oracle(order, records):
    """A plan large enough to set items aside, without and with streams of records."""
    import torch

    import paper_2106_12863_amd as sinet
    rng = np.random.default_rng(8)
    base, plen = rng.integers(0, 1 << 32, 64).astype(np.uint32), rng.integers(3, 20, 64).astype(np.uint8)
    tab = sinet.Table(base, plen)
    print("batch set aside", order, flush=True)
    made = [_stream(sinet, torch, tab, base, plen, 80, 15_000_007, 500, 20_000, order, True)]
    lab, out, exp = made[0][1:]
    s = made[0][0]
    extra = [sinet.new_hist(20_000) for _ in range(5)]  # the same sessions again, other outputs
    streams = [s] + [sinet.BatchStream(tab, s.ts, s.src, s.dst, s.nbytes, 300, 500, 20_000, out=o) for o in extra]
    made += [_stream(sinet, torch, tab, base, plen, 81, 300_001, 10, 70_000, order, True)] if records else []
    plan = sinet.BatchPlan(streams[:2] + [m[0] for m in made[1:]] + streams[2:])
    for _ in range(3):
        plan.run()
        torch.cuda.synchronize()
        assert np.array_equal(lab.cpu().numpy(), exp[0])
        for o in [out] + extra:
            for got, e in zip(o, exp[1:]):
                assert np.array_equal(sinet.to_host_u64(got), e)
        for _, _, o, e in made[1:]:
            assert all(np.array_equal(sinet.to_host_u64(a), b) for a, b in zip(o, e[1:]))


def test_coarse_streams_out_of_order_equal_oracle():
    import torch

    import paper_2106_12863_amd as sinet
    rng = np.random.default_rng(7)
    made = []
    for j, (kind, order, n, width, n_bins) in enumerate([
            ("scan", "shuffled", 400_009, 1_000, 3_000), ("auto", "half", 700_001, 1_000, 3_000),
            ("trie", "half", 600_011, 1_000, 20_000), ("auto", "shuffled", 1_200_007, 500, 65_536),
            ("scan", "half", 1_300_001, 500, 70_000),      # more bins than are set aside
            ("auto", "sorted", 300_001, 1_000, 5_000), ("scan", "shuffled", 50_001, 60_000, 60),
            ("auto", "shuffled", 200_003, 20, 30_000)]):   # records anyway
        k = 64 if kind == "scan" else 3_000
        base, plen = rng.integers(0, 1 << 32, k).astype(np.uint32), rng.integers(5, 29, k).astype(np.uint8)
        tab = sinet.Table(base, plen, kind=kind, inout_index=kind != "trie")
        made.append(_stream(sinet, torch, tab, base, plen, 50 + j, n, width, n_bins, order, j % 2 == 0))
    print("batch out of order", flush=True)
    for chunk in (None, 2_048, 1 << 18):
        tune = None
        if chunk:
            tune = sinet.Tune()
            tune.block, tune.chunk, tune.grid = 512, chunk, 0
        _check(sinet, torch, sinet.BatchPlan([m[0] for m in made], tune), made)
