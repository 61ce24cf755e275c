"""The lookup pass's search queues against the CPU oracle: waves (64 lanes of
four sessions, 512 addresses) in which given numbers of addresses lie in /16
blocks that prefixes cut, around the sizes of a round, of a pair step and of the
ring, for the kinds whose queued searches are read by pairs of lanes."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

SEARCHED = (0, 1, 2, 31, 32, 33, 63, 64, 65, 127, 128, 129, 191, 193, 320, 511, 512)


@pytest.mark.parametrize("kind,train", [("bsearch", None), ("trie", None), ("mlp", dict(steps=50)),
                                        ("pla", dict(target_err=2)), ("pla", dict(target_err=6)),
                                        ("pla", dict(segments=8))])
@pytest.mark.parametrize("prefixes", [40, 9_000])
def test_queued_labels_equal_oracle(prefixes, kind, train):
    import torch

    import paper_2106_12863_amd as sinet
    rng = np.random.default_rng(11)
    plen = rng.integers(18, 33, prefixes).astype(np.uint8)
    base = rng.integers(0, 1 << 32, prefixes).astype(np.uint32)
    tab = sinet.Table(base, plen, kind=kind, inout_index=False)
    if train:
        tab.train(**train)
    low = (np.uint64(0xFFFFFFFF) << (32 - plen).astype(np.uint64)).astype(np.uint32)
    edges = np.concatenate([base & low, (base & low) - np.uint32(1), base | ~low, (base | ~low) + np.uint32(1)])
    cut = np.unique(base >> 16)
    free = np.setdiff1d(np.arange(1 << 16, dtype=np.uint32), cut)
    waves = []
    for k in SEARCHED:
        inside = (rng.choice(cut, 512) << 16) | rng.integers(0, 1 << 16, 512).astype(np.uint32)
        edge = rng.choice(edges, 512)
        inside = np.where((rng.random(512) < 0.5) & np.isin(edge >> 16, cut), edge, inside)
        outside = (rng.choice(free, 512) << 16) | rng.integers(0, 1 << 16, 512).astype(np.uint32)
        hit = np.zeros(512, bool)
        hit[rng.permutation(512)[:k]] = True
        waves.append(np.where(hit, inside, outside).astype(np.uint32).reshape(2, 256))
    ends = np.tile(np.concatenate(waves, axis=1), (1, 40))
    for n in (1, 256, 257, 256 * len(SEARCHED), ends.shape[1] - 3):
        src, dst = ends[:, :n]
        exp = oracle.classify(base, plen, src, dst)[0]
        print("search queue", prefixes, kind, train, n, flush=True)
        lab = sinet.discriminate(tab, sinet.to_device_u32(src), sinet.to_device_u32(dst))[0]
        torch.cuda.synchronize()
        assert np.array_equal(lab.cpu().numpy(), exp)
