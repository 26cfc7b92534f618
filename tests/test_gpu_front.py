"""The pass that packs the input and marks valid windows, where it can go wrong:
reads at every alignment, inputs that end about a 64-byte chunk or about a
workgroup's 255 or 254 chunks, windows over that line, read ends in any place,
many empty reads at one. Against the oracle, bit-exact."""
import numpy as np
import pytest

import oracle
from gpu_util import assert_same, gpu_count

pytestmark = pytest.mark.gpu


def _bases(n, seed):
    rng = np.random.default_rng(seed)
    r = np.frombuffer(b"ACGTacgt", dtype=np.uint8)[rng.integers(0, 8, n)].copy()
    r[rng.integers(0, n, 1 + n // 900)] = ord("N")
    return r, rng


@pytest.mark.parametrize("n", [1, 63, 64, 65, 255 * 64 - 1, 255 * 64 + 1, 254 * 64, 256 * 64,
                               2 * 255 * 64 + 17])
@pytest.mark.parametrize("pad", [0, 1, 3, 16, 21])
def test_alignment_and_ends(n, pad):
    r, rng = _bases(n, n + pad)
    cuts = np.sort(rng.integers(0, n + 1, n // 300))
    cuts = np.concatenate([cuts, [c for c in (64, 254 * 64, 255 * 64, 256 * 64 - 1) if c <= n]])
    o = np.concatenate([[0], np.sort(cuts), [n]]).astype(np.uint64)
    for k in (1, 31, 64, 65, 128):
        assert_same(gpu_count(r, o, k, P=2, pad_front=pad), oracle.count(r, o, k),
                    "%d bytes from %d, k %d" % (n, pad, k))


@pytest.mark.parametrize("empty", [1, 1023, 1024, 1025, 5000])
def test_empty_reads(empty):
    n = 40_000
    r, _ = _bases(n, empty)
    # reads of one length, as many empty ones at the start, in two places and at the end
    o = np.concatenate([np.arange(0, n, 97)] + [np.full(empty, p) for p in (0, 9700, 9797, n)] + [[n]])
    o = np.sort(o).astype(np.uint64)
    for k in (31, 100):
        assert_same(gpu_count(r, o, k), oracle.count(r, o, k), "%d empty reads, k %d" % (empty, k))


def test_unequal_reads():
    # reads of very unequal lengths: their ends are far from where equal lengths would have them
    n = 300_000
    r, _ = _bases(n, 5)
    o = np.unique(np.concatenate([np.arange(0, 60_000, 3), [n // 2, n]])).astype(np.uint64)
    for k in (3, 31):
        assert_same(gpu_count(r, o, k, P=4), oracle.count(r, o, k), "k %d" % k)
