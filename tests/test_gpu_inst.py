"""Institution ids through the institution index against the CPU oracle: few
institutions (codes in the leaves) and more than the codes take, a table whose
records and samples do not fit LDS, many leaves in one /16 block, ragged sizes,
unaligned columns and outputs, and several sets of requested outputs."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _table(shape):
    rng = np.random.default_rng(7)
    if shape == "hosts":       # 400 hosts inside one /23
        base = (0x0A0B0000 + rng.choice(512, 400, replace=False)).astype(np.uint32)
        plen = np.full(400, 32, np.uint8)
    elif shape == "wide":      # every /16 block cut, more than 65,536 leaves
        plen = rng.integers(18, 29, 200_000).astype(np.uint8)
        base = rng.integers(0, 1 << 32, 200_000).astype(np.uint32)
    else:                      # everything covered, nested
        plen = np.concatenate([[0, 1], rng.integers(4, 33, 9_000)]).astype(np.uint8)
        base = rng.integers(0, 1 << 32, 9_002).astype(np.uint32)
    if shape.endswith("rows"):  # one institution per row: no codes
        return base, plen, np.arange(len(base), dtype=np.uint32)
    return base, plen, rng.integers(0, 500, len(base)).astype(np.uint32)


@pytest.mark.parametrize("shape", ["hosts", "wide", "cover", "cover_rows"])
def test_institutions_equal_oracle(shape):
    import torch

    import paper_2106_12863_amd as sinet
    base, plen, inst = _table(shape)
    rng = np.random.default_rng(8)
    tab = sinet.Table(base, plen, inst)
    for n, off in ((1, 0), (3, 1), (2_051, 0), (70_003, 3), (300_000, 0)):
        print("institutions", shape, n, off, flush=True)
        end = rng.integers(0, 1 << 32, (2, n + off)).astype(np.uint32)
        pick = rng.integers(0, len(base), (2, n + off))
        near = base[pick] + rng.integers(-3, 600, (2, n + off)).astype(np.uint32)
        a = np.where(rng.random((2, n + off)) < 0.6, near, end)
        src, dst = (sinet.to_device_u32(x)[off:] for x in a)
        lab, si, di = oracle.classify(base, plen, a[0][off:], a[1][off:], inst)
        for want in ((1, 1, 1), (0, 1, 0), (1, 0, 1)):
            out = [torch.full((n + 1,), 7, dtype=t, device="cuda")[1:] if off == 3 else
                   torch.full((n,), 7, dtype=t, device="cuda")
                   for t in (torch.uint8, torch.int32, torch.int32)]
            got = sinet.discriminate(tab, src, dst, *[o if w else False for o, w in zip(out, want)])
            torch.cuda.synchronize()
            for g, e, w in zip(got, (lab, si, di), want):
                assert (g is not None) == bool(w)
                if w:
                    assert np.array_equal(g.cpu().numpy().view(e.dtype), e), (n, want)
