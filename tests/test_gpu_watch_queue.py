"""The watch kernel's collected searches against the CPU oracle: lists that let
no, few, many or all addresses through the /16 filter, so that a wave's queue
fills in every round, over iterations, or only at the end."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("share", ["none", "few", "many", "all"])
@pytest.mark.parametrize("kind", ["bsearch", "trie"])
def test_watch_queue_equals_oracle(share, kind):
    import torch

    import paper_2106_12863_amd as sinet
    rng = np.random.default_rng(4)
    if share == "all":
        base, plen = np.array([0, 0x80000000, 0x80000000], np.uint32), np.array([1, 1, 9], np.uint8)
    elif share == "many":
        base, plen = rng.integers(0, 1 << 32, 300).astype(np.uint32), rng.integers(6, 33, 300).astype(np.uint8)
    else:
        base, plen = rng.integers(0, 1 << 32, 200).astype(np.uint32), np.full(200, 32, np.uint8)
    keys = rng.integers(0, 7, len(base)).astype(np.uint32)
    tab = sinet.Table(base, plen, keys, kind=kind)
    for n in (1, 255, 2_049, 1_700_003):  # the last: more than one iteration
        ends = rng.integers(0, 1 << 32, (2, n)).astype(np.uint32)
        if share != "none":
            ends = np.where(rng.random((2, n)) < 0.05, rng.choice(base, (2, n)), ends)
        ts = rng.integers(0, 100_000, n).astype(np.uint32)
        by = rng.integers(0, 1 << 40, n).astype(np.uint64)
        exp = oracle.watch(base, plen, ts, ends[0], ends[1], by, 500, 777, 100, 7, inst=keys)
        for off in (0, 1):
            print("watch queue", share, kind, n, off, flush=True)
            pad = [np.concatenate([a[:off], a]) for a in (ts, ends[0], ends[1], by)]
            d = [sinet.to_device_u32(a)[off:] for a in pad[:3]] + [sinet.to_device_u64(pad[3])[off:]]
            out = sinet.watch_histogram(tab, *d, 500, 777, 100, 7)
            torch.cuda.synchronize()
            for got, e in zip(out, exp):
                assert np.array_equal(sinet.to_host_u64(got).reshape(e.shape), e)
