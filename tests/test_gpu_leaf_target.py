"""Leaves of two-word keys whose records are all distinct (random reads) mostly fit
their first table."""
import numpy as np
import pytest

import oracle
import paper_2505_04431_amd as kc
from gpu_util import assert_same, gpu_count

pytestmark = pytest.mark.gpu

TARGET, LIMIT = 1920, 1792  # records of a leaf; distinct keys at which its table gives up


def _reads(n, seed):
    rng = np.random.default_rng(seed)
    r = np.frombuffer(b"ACGT", dtype=np.uint8)[rng.integers(0, 4, n)].copy()
    return r, np.concatenate([np.arange(0, n, 150), [n]]).astype(np.uint64)


@pytest.mark.parametrize("k", [33, 55, 64])
def test_all_distinct(k):
    share = []
    for mb in (1.3, 1.8, 2.5, 3.5, 4, 5, 6, 7, 9, 11, 14):
        r, o = _reads(int(mb * 1e6), int(mb * 10) + k)
        got = gpu_count(r, o, k, P=64)
        s = kc.last_stats()
        share.append(s["second_records"] / s["valid_windows"])
        if mb in (1.3, 6):
            assert_same(got, oracle.count(r, o, k), "k %d, %g MB" % (k, mb))
    # shards are cut in powers of two, so leaves lie between half the target and the
    # target; spread evenly, this share of their records is in those above the limit
    assert np.mean(share) <= (TARGET**2 - LIMIT**2) / (TARGET**2 - (TARGET / 2)**2), share
