"""The kinds' own searches where a table has no index: institution ids through
every kind's lookup, and scan tables' labels by the row scan, on aligned and
offset columns, against the CPU oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _prefixes(rng, kind):
    n = 64 if kind == "scan" else 6_000
    base = rng.integers(0, 1 << 32, n).astype(np.uint32)
    plen = rng.integers(4 if kind == "scan" else 12, 31, n).astype(np.uint8)
    base[:3], plen[:3] = (0, 0xFFFFFFFF, 0x80000000), (9, 32, 32)
    return base, plen, rng.integers(0, 1 << 31, n).astype(np.uint32)


def _addresses(rng, base, n):
    near = base[rng.integers(0, len(base), (2, n))] + rng.integers(-2, 400, (2, n))
    return np.where(rng.random((2, n)) < 0.6, near, rng.integers(0, 1 << 32, (2, n))).astype(np.uint32)


def _table(sinet, kind, base, plen, inst):
    tab = sinet.Table(base, plen, inst, kind=kind.split("_")[0], inout_index=False,
                      global_bsearch=kind == "bsearch_global") if kind != "pla_wide" else \
        sinet.Table(base, plen, inst, kind="pla", inout_index=False)
    if kind.startswith("pla"):
        tab.train(segments=100 if kind == "pla_wide" else 0)
    elif kind == "mlp":
        tab.train(steps=30)
    return tab


@pytest.mark.parametrize("kind", ["scan", "bsearch", "bsearch_global", "trie", "pla", "pla_wide", "mlp"])
def test_institutions_by_the_kinds_search(kind):
    import torch

    import paper_2106_12863_amd as sinet
    rng = np.random.default_rng(len(kind))
    base, plen, inst = _prefixes(rng, kind)
    tab = _table(sinet, kind, base, plen, inst)
    for n, off in ((1, 0), (5, 1), (4_099, 0), (60_003, 3), (300_000, 0)):
        print("institutions by", kind, n, off, flush=True)
        a = _addresses(rng, base, n + off)
        src, dst = (sinet.to_device_u32(x)[off:] for x in a)
        lab, si, di = oracle.classify(base, plen, a[0][off:], a[1][off:], inst)
        for want in ((1, 1, 1), (0, 0, 1), (1, 1, 0)):
            out = [torch.full((n + off,), 7, dtype=t, device="cuda")[off:]
                   for t in (torch.uint8, torch.int32, torch.int32)]
            got = sinet.discriminate(tab, src, dst, *[o if w else False for o, w in zip(out, want)])
            torch.cuda.synchronize()
            for g, e, w in zip(got, (lab, si, di), want):
                assert (g is not None) == bool(w)
                if w:
                    assert np.array_equal(g.cpu().numpy().view(e.dtype), e), (n, want)


@pytest.mark.parametrize("kind", ["bsearch", "trie", "pla", "mlp"])
@pytest.mark.parametrize("ids,deep", [(900, False), (1 << 30, False), (900, True)])
def test_institutions_of_tables_beyond_lds(kind, ids, deep):
    """Default tables whose index does not fit LDS: some kinds search themselves."""
    import torch

    import paper_2106_12863_amd as sinet
    rng = np.random.default_rng(ids % 1000)
    base = (rng.integers(0, 1 << 24, 70_000) << 8).astype(np.uint32)
    plen = np.full(70_000, 24, np.uint8)
    if deep:  # 600,000 hosts in 2,000 blocks: many groups in a block
        base = ((rng.integers(0, 2_000, 600_000) * 32 << 16) + rng.integers(0, 1 << 16, 600_000)).astype(np.uint32)
        base, plen = base[:250_000], np.full(250_000, 32, np.uint8)
    inst = rng.integers(0, ids, len(base)).astype(np.uint32)
    tab = sinet.Table(base, plen, inst, kind=kind)
    if kind in ("pla", "mlp"):
        tab.train(steps=30 if kind == "mlp" else 0)
    n = 200_003
    print("institutions beyond LDS", kind, ids, flush=True)
    a = _addresses(rng, base, n)
    got = sinet.discriminate(tab, *(sinet.to_device_u32(x) for x in a), True, True, True)
    torch.cuda.synchronize()
    for g, e in zip(got, oracle.classify(base, plen, a[0], a[1], inst)):
        assert np.array_equal(g.cpu().numpy().view(e.dtype), e)


@pytest.mark.parametrize("n,width,n_bins", [(3, 1, 5_000), (300_007, 1, 5_000), (300_007, 50, 100),
                                            (400_003, 60, 4_000), (400_003, 9, 4_000)])
def test_scan_labels_by_the_row_scan(n, width, n_bins):
    """Records, whole and moving windows, and the order probe."""
    import torch

    import paper_2106_12863_amd as sinet
    rng = np.random.default_rng(n + width)
    base, plen, inst = _prefixes(rng, "scan")
    tab = _table(sinet, "scan", base, plen, inst)
    ts = (np.sort(rng.integers(0, n_bins * width + 50, n)) + 7).astype(np.uint32)
    by = rng.integers(0, 1 << 40, n).astype(np.uint64) >> rng.integers(0, 40, n).astype(np.uint64)
    a = _addresses(rng, base, n)
    exp = oracle.pipeline(base, plen, ts, a[0], a[1], by, 7, width, n_bins)
    for off in (0, 1):
        print("row scan", n, width, n_bins, off, flush=True)
        c = [sinet.to_device_u32(np.concatenate([x[:off], x]))[off:] for x in (ts, a[0], a[1])]
        c.append(sinet.to_device_u64(np.concatenate([by[:off], by]))[off:])
        lab, out = sinet.pipeline(tab, *c, 7, width, n_bins)
        only = sinet.discriminate(tab, c[1], c[2])[0]
        torch.cuda.synchronize()
        assert np.array_equal(lab.cpu().numpy(), exp[0]) and torch.equal(lab, only)
        for got, e in zip(out, exp[1:]):
            assert np.array_equal(sinet.to_host_u64(got), e)
