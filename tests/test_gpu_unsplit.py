"""Inputs counted without a split: sizes about the line (1,024 bytes a shard for
one-word keys, 512 for wider ones), shards of far more records than the others, and of more
distinct keys than the table holds (counted again with a split). Against the
oracle, bit-exact."""
import numpy as np
import pytest

import oracle
import paper_2505_04431_amd as kc
from gpu_util import assert_same, gpu_count

pytestmark = pytest.mark.gpu


def _reads(n, letters, seed):
    rng = np.random.default_rng(seed)
    r = np.frombuffer(letters, dtype=np.uint8)[rng.integers(0, len(letters), n)].copy()
    o = np.unique(np.concatenate([np.arange(0, n, 151), [n]])).astype(np.uint64)
    return r, o


@pytest.mark.parametrize("n", [60, 2_048, 40_000, 131_072, 131_073, 262_144, 262_145])
@pytest.mark.parametrize("k", [1, 4, 5, 21, 32, 33, 64, 65, 100])
def test_about_the_line(n, k):
    r, o = _reads(n, b"ACGT", n + k)
    for P in (1, 300):
        assert_same(gpu_count(r, o, k, P=P, check=1), oracle.count(r, o, k),
                    "%d bytes, k %d, P %d" % (n, k, P))


@pytest.mark.parametrize("k", [13, 21, 31, 32, 40, 64, 90])
@pytest.mark.parametrize("letters", [b"AT", b"AAAAAAAT", b"AAAAAAAC", b"CG", b"A", b"AAAATTTTCG"])
def test_unequal_shards(k, letters):
    r, o = _reads(262_000 if k <= 32 else 131_000, letters, 3)
    got = gpu_count(r, o, k, check=1)
    assert_same(got, oracle.count(r, o, k), "k %d, %s" % (k, letters))
    assert kc.last_stats()["valid_windows"] == int(got[1].sum())
