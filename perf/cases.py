"""Workloads that time libsinet through its public entry points.

``listed()`` names the workloads, ``draw(rng)`` gives one more of the same
ranges, ``prepare(case, seed)`` makes what a program holds before the call
(resident columns, tables, plans, output buffers), ``run(state)`` is one pass
and ``work(case)`` the bytes it cannot do without.  Inputs are synthetic and
SINET-shaped: nearly time-sorted sessions (diurnal rate, +-5 s jitter), 30% of
the addresses inside the prefix table, lognormal byte counts.  Every output is
a whole number or a byte, so ``exact`` has nothing to add.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2106_12863_amd as sinet

DAY_MS = 86_400_000
ORIGIN_DAYS = 18_677  # 2021-02-19


# ---------------------------------------------------------------------------
# the workloads
# ---------------------------------------------------------------------------
def listed():
    return [
        # A live feed handed over in small chunks: per-second counts of ten
        # thousand sessions of one minute; launches and latency count.
        dict(name="chunk_1e4_seconds", op="pipeline", n=10_000, span=60_000, width=1_000,
             table="tiny", label=True),
        # One minute of traffic at full resolution against a small table.
        dict(name="minute_1e6_ms", op="pipeline", n=1_000_000, span=60_000, width=1,
             table="tiny", label=True),
        # A day of a mid-size network in millisecond bins.
        dict(name="day_1e8_ms", op="pipeline", n=100_000_000, span=DAY_MS, width=1,
             table="nested", label=True),
        # The whole backbone's day (Table 2's 1.6 billion sessions) against
        # 200,000 prefixes in millisecond bins.
        dict(name="fullday_16e8_ms", op="pipeline", n=1_600_000_000, span=DAY_MS, width=1,
             table="clustered", label=True),
        # A day in one-second bins (a monitoring plot), no labels kept.
        dict(name="day_1e8_seconds", op="pipeline", n=100_000_000, span=DAY_MS, width=1_000,
             table="clustered", label=False),
        # Sessions labelled earlier, counted into the paper's ten-minute frames.
        dict(name="frames_4e8_tenmin", op="histogram", n=400_000_000, span=DAY_MS, width=600_000),
        # 64 uneven streams, each with its own table, window and bin width.
        dict(name="batch_64_streams", op="batch", streams=64, n=300_000_000),
        # Longest-match institution of both ends of every session.
        dict(name="institutions_1e8", op="institutions", n=100_000_000, table="clustered",
             kind="auto"),
        # Labels through the learned index (no in/out index), 5e8 sessions.
        dict(name="learned_5e8_labels", op="labels", n=500_000_000, table="clustered", kind="pla"),
        # Two watch lists (300 + 877 hosts) over a day in ten-minute frames.
        dict(name="watch_4e8_tenmin", op="watch", n=400_000_000, hosts=1_177, span=DAY_MS,
             width=600_000),
        # A text chunk of the session log (about 200 bytes a line) to columns.
        dict(name="parse_2e7_lines", op="parse", n=20_000_000),
        # Millisecond bins of a day summed to one-hour frames.
        dict(name="rebin_day_hours", op="rebin", rows=4, n_bins=DAY_MS, factor=3_600_000),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["pipeline", "pipeline", "pipeline", "histogram", "batch", "institutions",
                     "labels", "watch", "parse", "rebin"])
    if op == "pipeline":
        span = _log(rng, 60_000, DAY_MS)
        return dict(op=op, n=_log(rng, 5_000, 200_000_000), span=span,
                    width=rng.choice([1, 1, 10, 1_000, 1_000, 60_000]),
                    table=rng.choice(["tiny", "nested", "clustered"]), label=rng.random() < 0.7)
    if op == "histogram":
        span = _log(rng, 3_600_000, DAY_MS)
        return dict(op=op, n=_log(rng, 100_000, 400_000_000), span=span,
                    width=rng.choice([1, 10, 1_000, 60_000, 600_000, 3_600_000]))
    if op == "batch":
        k = rng.randint(2, 64)
        return dict(op=op, streams=k, n=_log(rng, 10_000 * k, 4_000_000 * k))
    if op in ("institutions", "labels"):
        return dict(op=op, n=_log(rng, 10_000, 200_000_000),
                    table=rng.choice(["nested", "clustered"]),
                    kind=rng.choice(["auto", "auto", "trie", "pla", "mlp"]))
    if op == "watch":
        span = _log(rng, 3_600_000, DAY_MS)
        return dict(op=op, n=_log(rng, 100_000, 400_000_000), hosts=rng.randint(50, 2_000),
                    span=span, width=rng.choice([60_000, 600_000, 3_600_000]))
    if op == "parse":
        return dict(op=op, n=_log(rng, 1_000, 20_000_000))
    return dict(op=op, rows=4, n_bins=_log(rng, 60_000, DAY_MS),
                factor=rng.choice([10, 60, 1_000, 60_000, 600_000, 3_600_000]))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _rng(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g, np.random.Generator(np.random.PCG64(seed))


def _masks(plen):
    return np.where(plen == 0, 0, (0xFFFFFFFF << (32 - plen.astype(np.int64))) & 0xFFFFFFFF)


def _nest(rng, base, plen, k, lmax, extra):
    """k more prefixes, each strictly inside one of the given ones."""
    cand = np.flatnonzero(plen < lmax)
    par = cand[rng.integers(0, len(cand), k)]
    hi = np.minimum(lmax, plen[par] + extra)
    ln = plen[par] + 1 + (rng.random(k) * (hi - plen[par])).astype(np.int64)
    host = rng.integers(0, 1 << 32, k) & ~_masks(plen[par]) & 0xFFFFFFFF
    return (np.concatenate([base, (base[par] | host) & _masks(ln)]),
            np.concatenate([plen, ln]))


def _nested_table(rng, n, lmin, lmax, frac):
    k = int(round(n * frac))
    plen = rng.integers(lmin, lmax + 1, n - k)
    base = rng.integers(0, 1 << 32, n - k) & _masks(plen)
    return _nest(rng, base, plen, k, lmax, lmax) if k else (base, plen)


def _clustered_table(rng, n=200_000, frac=0.3):
    """Consecutive aligned sub-prefixes in allocation blocks (lognormal block
    sizes, lengths 8..32 peaked at /24), a share of them nested further."""
    top = n - int(round(n * frac))
    ls = np.arange(8, 33)
    w = np.exp(-np.abs(ls - 24) / 2.0)
    blocks = top // 16
    ln = rng.choice(ls, blocks, p=w / w.sum())
    c = np.clip(np.rint(np.exp(rng.normal(math.log(20.0), 1.0, blocks))), 1, 4096).astype(np.int64)
    c = np.where(ln < 16, 1, c)
    bits = np.minimum(np.ceil(np.log2(c)).astype(np.int64), ln)
    start = rng.integers(0, 1 << 32, blocks) & _masks(ln - bits)
    own = np.repeat(np.arange(blocks), c)
    slot = np.arange(len(own)) - np.repeat(np.cumsum(c) - c, c)
    base = (start[own] + (slot << (32 - ln[own]))) & 0xFFFFFFFF
    base, plen = _nest(rng, base[:top], ln[own][:top], n - min(top, len(own)), 32, 8)
    p = rng.permutation(len(base))
    return base[p], plen[p]


def _prefixes(rng, table):
    if table == "tiny":
        base, plen = _nested_table(rng, 64, 16, 24, 0.0)
    elif table == "nested":
        base, plen = _nested_table(rng, 1_024, 12, 28, 0.2)
    else:
        base, plen = _clustered_table(rng)
    return base.astype(np.uint32), plen.astype(np.uint8)


def _day_knots():
    """Inverse of the diurnal distribution (rate 1 - cos/2 over a day)."""
    x = np.linspace(0.0, 1.0, 8193)
    return np.interp(np.linspace(0.0, 1.0, 4097), x - np.sin(2 * np.pi * x) / (4 * np.pi), x)


def _columns(g, n, span, prefixes, only=("ts", "src", "dst", "bytes"), hosts=None):
    """Resident session columns (uint32 in int32, uint64 in int64 tensors)."""
    dt = dict(ts=torch.int32, src=torch.int32, dst=torch.int32, bytes=torch.int64)
    out = {k: torch.empty(n, dtype=dt[k], device="cuda") for k in only}
    base, plen = prefixes
    tb = torch.from_numpy(base.view(np.int32).copy()).cuda()
    th = torch.from_numpy((~_masks(plen) & 0xFFFFFFFF).astype(np.uint32).view(np.int32)).cuda()
    knots = torch.from_numpy(_day_knots()).cuda()
    jit = min(5_000, span // 20)
    step = 1 << 25
    for a in range(0, n, step):
        m = min(step, n - a)
        if "ts" in out:
            u = (torch.arange(a, a + m, device="cuda", dtype=torch.float64) + 0.5) * (4096.0 / n)
            k = u.to(torch.int64).clamp_(max=4095)
            t = torch.lerp(knots[k], knots[k + 1], u - k) * span
            t = t.to(torch.int64) + torch.randint(-jit, jit + 1, (m,), generator=g, device="cuda")
            t = torch.where(t < 0, -t - 1, t)
            out["ts"][a:a + m] = torch.where(t >= span, 2 * span - 1 - t, t).to(torch.int32)
            del u, k, t
        for c in ("src", "dst"):
            if c in out:
                r = torch.randint(-(1 << 31), 1 << 31, (m,), generator=g, device="cuda",
                                  dtype=torch.int32)
                p = torch.randint(0, len(base), (m,), generator=g, device="cuda",
                                  dtype=torch.int32)
                inside = torch.rand(m, generator=g, device="cuda") < 0.3
                r = torch.where(inside, tb[p] | (r & th[p]), r)
                if hosts is not None:  # 0.2% of each end is a listed host, a few of them often
                    hit = torch.rand(m, generator=g, device="cuda") < 0.002
                    v = torch.rand(m, generator=g, device="cuda").square_().mul_(len(hosts))
                    r = torch.where(hit, hosts[v.to(torch.int32).clamp_(max=len(hosts) - 1)], r)
                out[c][a:a + m] = r
                del r, p, inside
        if "bytes" in out:
            z = torch.empty(m, device="cuda").normal_(8.0, 2.0, generator=g)
            out["bytes"][a:a + m] = z.exp_().clamp_(1.0, 5e7).to(torch.int64)
    return out


def _bins(case):
    return -(-case["span"] // case["width"])


def _table(rng, table, kind, inout=True):
    base, plen = _prefixes(rng, table)
    inst = rng.integers(0, 1_000, len(base)).astype(np.uint32)
    t = sinet.Table(base, plen, inst, kind=kind, inout_index=inout)
    if kind in ("pla", "mlp"):
        t.train(steps=200 if kind == "mlp" else 0)
    return t, (base, plen)


_COUNTRY = [b"JP", b"US", b"CN", b"KR", b"DE", b"GB", b"FR", b"NL", b"SG"]
_APP = [b"ssl", b"web-browsing", b"dns", b"ntp", b"quic", b"ssh", b"smtp", b"incomplete"]
_REASON = [b"tcp-fin", b"aged-out", b"tcp-rst-from-client", b"policy-deny"]
_CATEGORY = [b"any", b"computer-and-internet-info", b"search-engines"]


def _text(g, n):
    """n lines of the 24-field session record (one flat uint8 tensor)."""
    parts = []
    for a in range(0, n, 1 << 20):
        m = min(1 << 20, n - a)
        chars, keep = [], []

        def put(c, k):
            chars.append(c)
            keep.append(k)

        def lit(s):
            t = torch.tensor(list(s), dtype=torch.uint8, device="cuda")
            put(t.expand(m, len(s)), torch.ones((m, len(s)), dtype=torch.bool, device="cuda"))

        def num(x, width, pad=False):
            p = 10 ** torch.arange(width - 1, -1, -1, device="cuda", dtype=torch.int64)
            q = x[:, None] // p
            k = q > 0
            k[:, -1] = True
            put((q % 10 + 48).to(torch.uint8), torch.ones_like(k) if pad else k)

        def pick(words):
            w = max(map(len, words))
            t = torch.tensor([list(s.ljust(w, b"\0")) for s in words], dtype=torch.uint8,
                             device="cuda")
            c = t[rnd(len(words))]
            put(c, c > 0)

        def rnd(hi, lo=0):
            return torch.randint(lo, hi, (m,), generator=g, device="cuda")

        def when(ms, milli=False):
            lit(b"2021/02/19 ")
            for div, mod, end in ((3_600_000, 24, b":"), (60_000, 60, b":"), (1_000, 60, b"")):
                num(ms // div % mod, 2, True)
                if end:
                    lit(end)
            if milli:
                lit(b".")
                num(ms % 1_000, 3, True)

        def addr():
            for k in range(4):
                num(rnd(256), 3)
                lit(b"." if k < 3 else b",")

        ms = ((torch.arange(a, a + m, device="cuda", dtype=torch.float64) + 0.5) *
              (0.98 * DAY_MS / n)).to(torch.int64) + rnd(10_000)
        size = torch.empty(m, device="cuda").normal_(8.0, 2.0, generator=g).exp_() \
            .clamp_(1.0, 5e7).to(torch.int64)
        took = rnd(600)
        when(ms, True)
        lit(b",")
        when(ms)
        lit(b",")
        when((ms - took * 1_000).clamp_(min=0))
        lit(b",")
        num(took, 3)
        lit(b",")
        addr()
        num(rnd(65_536), 5)
        lit(b",")
        pick(_COUNTRY)
        lit(b",")
        addr()
        num(rnd(65_536), 5)
        lit(b",")
        pick(_COUNTRY)
        lit(b",")
        pick([b"tcp", b"udp", b"icmp"])
        lit(b",")
        pick(_APP)
        lit(b",")
        pick([b"end", b"start", b"drop", b"deny"])
        lit(b",")
        pick([b"allow", b"deny", b"drop", b"reset-both"])
        lit(b",")
        pick(_REASON)
        lit(b",")
        num(rnd(4), 1)
        lit(b",")
        pick(_CATEGORY)
        lit(b",")
        packets = size // 900 + 1
        sent = packets * rnd(100) // 100
        for x in (packets, sent, packets - sent):
            num(x, 5)
            lit(b",")
        num(size, 8)
        lit(b",")
        out = size * rnd(100) // 100
        num(out, 8)
        lit(b",")
        num(size - out, 8)
        lit(b",PA-7080\n")
        parts.append(torch.cat(chars, 1)[torch.cat(keep, 1)])
    return torch.cat(parts)


def _batch(case, g, rng):
    k = case["streams"]
    inputs, rng = rng, np.random.Generator(np.random.PCG64([k, case["n"]]))  # sizes: the case's own
    sz = np.exp(rng.normal(math.log(2.5e6), 1.2, k))
    for _ in range(8):
        sz = np.clip(sz * (case["n"] / sz.sum()), 1e4, 2e7)
    sizes, shapes = [int(n) for n in sz], []
    budget = 3.1e8 / 64 * k  # bins of all streams together
    for _ in sizes:
        span = int(round(math.exp(rng.uniform(math.log(6e4), math.log(DAY_MS)))))
        width = int(rng.choice([1, 10, 1_000]))
        bins = -(-span // width)
        if bins > budget:
            width, bins = 1_000, -(-span // 1_000)
        budget -= bins
        shapes.append((span, width, bins))
    # the streams' outputs side by side in four buffers, each starting on 512 bytes
    lab = torch.zeros(sum(-(-n // 512) * 512 for n in sizes), dtype=torch.uint8, device="cuda")
    cnt, byt = (torch.zeros(sum(-(-4 * b // 64) * 64 for _, _, b in shapes), dtype=torch.int64,
                            device="cuda") for _ in range(2))
    drp = torch.zeros((k, 64), dtype=torch.int64, device="cuda")
    streams, at, ab = [], 0, 0
    for j, (n, (span, width, bins)) in enumerate(zip(sizes, shapes)):
        pfx = int(round(math.exp(rng.uniform(math.log(64), math.log(4096)))))
        base, plen = _nested_table(inputs, pfx, 8, 28, 0.2)
        base, plen = base.astype(np.uint32), plen.astype(np.uint8)
        c = _columns(g, n, span, (base, plen))
        streams.append(sinet.BatchStream(
            sinet.Table(base, plen), c["ts"], c["src"], c["dst"], c["bytes"], 0, width, bins,
            label=lab[at:at + n],
            out=(cnt[ab:ab + 4 * bins], byt[ab:ab + 4 * bins], drp[j, :8])))
        at += -(-n // 512) * 512
        ab += -(-4 * bins // 64) * 64
    return sinet.BatchPlan(streams), (lab, cnt, byt, drp)


def prepare(case, seed):
    g, rng = _rng(seed)
    op = case["op"]
    st = dict(op=op, case=case)
    if op == "pipeline":
        st["table"], pfx = _table(rng, case["table"], "auto")
        st["cols"] = _columns(g, case["n"], case["span"], pfx)
        st["label"] = torch.empty(case["n"], dtype=torch.uint8, device="cuda") \
            if case["label"] else False
        st["out"] = sinet.new_hist(_bins(case))
    elif op == "histogram":
        st["cols"] = _columns(g, case["n"], case["span"], _prefixes(rng, "tiny"), ("ts", "bytes"))
        # three of ten ends inside: external 49%, egress and ingress 21% each, internal 9%
        lab = torch.empty(case["n"], dtype=torch.uint8, device="cuda")
        for a in range(0, case["n"], 1 << 26):
            m = min(1 << 26, case["n"] - a)
            s, d = (torch.rand(m, generator=g, device="cuda") < 0.3 for _ in range(2))
            lab[a:a + m] = s.to(torch.uint8) + 2 * d.to(torch.uint8)
        st["label"] = lab
        st["out"] = sinet.new_hist(_bins(case))
    elif op == "batch":
        st["plan"], st["out"] = _batch(case, g, rng)
    elif op in ("institutions", "labels"):
        st["table"], pfx = _table(rng, case["table"], case["kind"], op == "institutions")
        st["cols"] = _columns(g, case["n"], 1, pfx, ("src", "dst"))
        st["label"] = torch.empty(case["n"], dtype=torch.uint8, device="cuda")
        ids = op == "institutions"
        st["inst"] = [torch.empty(case["n"], dtype=torch.int32, device="cuda") if ids else False
                      for _ in range(2)]
    elif op == "watch":
        hosts = np.unique(rng.integers(0, 1 << 32, 2 * case["hosts"]))
        hosts = rng.permutation(hosts)[:case["hosts"]].astype(np.uint32)
        st["table"] = sinet.Table(hosts, np.full(len(hosts), 32, np.uint8))
        st["keys"] = len(hosts)
        st["cols"] = _columns(g, case["n"], case["span"], _prefixes(rng, "nested"),
                              hosts=torch.from_numpy(hosts.view(np.int32)).cuda())
        st["out"] = sinet.new_watch_hist(len(hosts), _bins(case))
    elif op == "parse":
        st["text"] = _text(g, case["n"])
    else:
        st["hist"] = torch.randint(0, 1 << 40, (case["rows"], case["n_bins"]), generator=g,
                                   device="cuda")
        st["out"] = torch.empty((case["rows"], -(-case["n_bins"] // case["factor"])),
                                dtype=torch.int64, device="cuda")
    torch.cuda.synchronize()
    return st


def run(st):
    op, case, c = st["op"], st["case"], st.get("cols")
    if op == "pipeline":
        lab, h = sinet.pipeline(st["table"], c["ts"], c["src"], c["dst"], c["bytes"], 0,
                                case["width"], _bins(case), label=st["label"], out=st["out"])
        return (*h, lab) if lab is not None else h
    if op == "histogram":
        return sinet.histogram(c["ts"], c["bytes"], st["label"], 0, case["width"], _bins(case),
                               out=st["out"])
    if op == "batch":
        st["plan"].run()
        return st["out"]
    if op in ("institutions", "labels"):
        r = sinet.discriminate(st["table"], c["src"], c["dst"], st["label"], *st["inst"])
        return [x for x in r if x is not None]
    if op == "watch":
        return sinet.watch_histogram(st["table"], c["ts"], c["src"], c["dst"], c["bytes"], 0,
                                     case["width"], _bins(case), st["keys"], out=st["out"])
    if op == "parse":
        cols, bad = sinet.parse_sessions(st["text"], ORIGIN_DAYS)
        return cols["ts"], cols["src"], cols["dst"], cols["bytes"], bad
    return sinet.rebin(st["hist"], case["factor"], out=st["out"])


def exact(case, seed):
    return None  # outputs are whole numbers and bytes


def work(case):
    op, n = case["op"], case.get("n", 0)
    if op == "pipeline":
        b = n * (20 + int(case["label"])) + 64 * _bins(case)
    elif op == "histogram":
        b = n * 13 + 64 * _bins(case)
    elif op == "batch":
        b = n * 21 + 64 * int(3.1e8 / 64 * case["streams"] * 0.8)
    elif op == "institutions":
        b = n * 17
    elif op == "labels":
        b = n * 9
    elif op == "watch":
        # both addresses, time and size of the sessions with a listed end, the cells
        b = n * 8 + int(n * 0.004) * 12 + 32 * case["hosts"] * _bins(case)
    elif op == "parse":
        b = n * (200 + 20)
    else:
        b = 8 * case["rows"] * (case["n_bins"] + -(-case["n_bins"] // case["factor"]))
    return {"bytes": b, "flops": 0}
