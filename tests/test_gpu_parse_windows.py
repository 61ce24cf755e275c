"""Session text around the edges of the parser's windows (32,768 bytes, of which
31,744 are owned) against the CPU oracle: newlines and field ends at every place
near an edge, windows with more newlines or delimiters than the lists hold, and
lines whose fields leave their window."""
import numpy as np
import pytest

import oracle
from sinetgen import text as stext

pytestmark = pytest.mark.gpu

OWN, WINDOW = 31_744, 32_768


def _line(rng, total=None, at=20):
    """A good line; with `total`, padded to that many bytes in field `at`."""
    f = ["2021/02/19 %02d:%02d:%02d.%03d" % tuple(int(rng.integers(0, k)) for k in (24, 60, 60, 1000))]
    f += ["x%d" % k for k in range(2, 21)]
    f[4], f[7] = (".".join(str(int(o)) for o in rng.integers(0, 256, 4)) for _ in range(2))
    f += [str(int(rng.integers(0, 10 ** int(rng.integers(1, 19))))), "s", "r", "PA"]
    if total is not None:
        f[at - 1] += "y" * (total - 1 - len(",".join(f)))
    return (",".join(f) + "\n").encode()


def _check(buf, off=0):
    import torch

    import paper_2106_12863_amd as sinet
    exp, ebad = oracle.parse(buf, stext.ORIGIN_DAYS)
    d = torch.from_numpy(np.concatenate([np.zeros(off, np.uint8), buf])).cuda()[off:]
    print("parse windows", len(buf), off, len(exp["ts"]), ebad, flush=True)
    cols, bad = sinet.parse_sessions(d, stext.ORIGIN_DAYS, capacity=len(exp["ts"]))
    torch.cuda.synchronize()
    assert bad == ebad and cols["ts"].shape[0] == len(exp["ts"])
    for k in ("ts", "src", "dst"):
        assert np.array_equal(sinet.to_host_u32(cols[k]), exp[k]), k
    assert np.array_equal(sinet.to_host_u64(cols["bytes"]), exp["bytes"])


def _fill(rng, n, parts):
    """Good lines up to exactly n bytes, then parts."""
    out, left = [], n
    while left > 1_000:
        out.append(_line(rng))
        left -= len(out[-1])
    if left:
        out.append(_line(rng, left) if left >= 200 else b"\n" * left)
    return np.frombuffer(b"".join(out) + b"".join(parts), np.uint8)


@pytest.mark.parametrize("edge", [OWN, WINDOW, 2 * OWN, OWN + WINDOW])
def test_newlines_near_an_edge(edge):
    rng = np.random.default_rng(edge)
    for d in (-200, -130, -64, -23, -2, -1, 0, 1, 2, 17, 64):
        buf = _fill(rng, edge + d, [_line(rng) for _ in range(300)])
        _check(buf, off=(d * 7) % 16)
        _check(buf[:edge + d], off=d % 5)      # the text ends here
        _check(buf[:edge + d - 1])             # ... without its newline


@pytest.mark.parametrize("what", ["short", "commas", "delims", "long", "digits"])
def test_lists_overflow_and_lines_leave_the_window(what):
    rng = np.random.default_rng(5)
    good = [_line(rng) for _ in range(150)]
    if what == "short":      # more than 1,024 newlines in a window, good lines among them
        mid = [b"\n" * 900, good[0], b"a\n" * 700, good[1], b",\n" * 2_000, good[2], b"\n" * 40_000]
    elif what == "commas":   # more than 6,144 delimiters before, inside and after good lines
        mid = [b"," * 6_100 + b"\n", good[0], good[1], good[2], good[3][:-1] + b"," * 30_000 + b"\n"]
    elif what == "delims":   # the list's end at every place of a good line
        mid = []
        for k in range(60):
            mid += [b"," * (6_100 + k) + b"\n", _line(rng), _line(rng), _line(rng)]
            size = sum(map(len, mid))
            mid.append(_line(rng, OWN * (k + 1) - size % (OWN * (k + 1))) if
                       OWN * (k + 1) - size >= 200 else b"")
    elif what == "long":     # the padded field leaves the window, before and after field 21
        mid = [_line(rng, n, at) for n in (1_500, 3_000, 33_000, 70_000) for at in (2, 9, 20, 24)]
        mid += [good[0][:-1] + b"z" * 200_000]
    else:                    # byte counts of 18 to 21 digits, octets and times out of range
        mid = [good[k % 150].replace(b",s,r,", b"%s,s,r," % x) for k, x in enumerate(
            [b"", b"0", b"00", b"000", b"0" * 12, b"x", b"-", b"\xb0"])]
        mid += [b"2021/02/19 00:00:00.000" + b"," * 4 + ip + b",p,c," + ip2 + b"," * 13 + n + b"\n"
                for ip in (b"1.2.3.4", b"255.255.255.255", b"256.1.1.1", b"1.2.3", b"1..2.3.4", b".1.2.3.4",
                           b"1.2.3.4.", b"0001.1.1.1", b"1.1.1.a", b"001.010.099.1")
                for ip2 in (b"9.8.7.6", b"1.2.3.4.5")
                for n in (b"1", b"18446744073709551615", b"18446744073709551616", b"9" * 19, b"9" * 21, b"", b"1 ")]
    buf = np.frombuffer(b"".join(good[:100] + mid + good[50:]), np.uint8)
    _check(buf)
    _check(buf[3:], off=11)


def test_bad_lines_are_counted_over_many_blocks():
    rng = np.random.default_rng(9)
    lines = [b"a" * int(k) + b"\n" for k in rng.integers(0, 90, 40_000)]
    for k in range(0, 40_000, 997):
        lines[k] = _line(rng)
    _check(np.frombuffer(b"".join(lines), np.uint8), off=5)


@pytest.mark.parametrize("at", [1, 2, 5, 9, 20, 21, 22, 24])
def test_one_line_beyond_its_window(at):
    """A last line that leaves its window by a field of every length around a step
    of the search (1,024 bytes), with and without a newline, cut after field 21,
    20 or 3, or with one field too long to be good."""
    rng = np.random.default_rng(at)
    head = _fill(rng, OWN - 150, []).tobytes()
    lines = []
    for n in (1_200, 2_040, 2_047, 2_048, 2_049, 5_000, 40_000):
        line = _line(rng, n + int(rng.integers(0, 16)), at)
        f = line[:-1].split(b",")
        lines += [line, b",".join(f[:21]) + b"\n", b",".join(f[:20]) + b"\n", b",".join(f[:3]) + b"\n",
                  b",".join(f[:20] + [b"18446744073709551615"] + f[21:]) + b"\n",
                  b",".join(f[:20] + [b"18446744073709551616"]) + b"\n"]
    for k, line in enumerate(lines):
        off = k % 16
        if k % 3 == 0:
            _check(np.frombuffer(head + line + _line(rng), np.uint8), off)
        elif k % 3 == 1:
            _check(np.frombuffer(head + line, np.uint8), off)
        else:
            _check(np.frombuffer(head + line[:-1], np.uint8), off)
