"""Which small inputs are counted without a split, told by the number of levels:
sizes on either side of the line, and inputs that a shard's distinct keys send to the
split after all. Against the oracle, bit-exact."""
import numpy as np
import pytest

import oracle
import paper_2505_04431_amd as kc
from gpu_util import assert_same, gpu_count

pytestmark = pytest.mark.gpu


def _reads(n, letters, seed):
    rng = np.random.default_rng(seed)
    r = np.frombuffer(letters, dtype=np.uint8)[rng.integers(0, len(letters), n)].copy()
    return r, np.concatenate([np.arange(0, n, 151), [n]]).astype(np.uint64)


# bytes a shard: 1,024 for one-word keys, 512 for wider ones; 256 shards up to P =
# 256, then 512 (where one-word keys are always split: the bound of their leaves
# that the host has is above the line for the larger table)
@pytest.mark.parametrize("k,P,line", [(13, 1, 1024 << 8), (31, 256, 1024 << 8), (32, 1, 1024 << 8),
                                      (33, 1, 512 << 8), (64, 64, 512 << 8), (100, 1, 512 << 8),
                                      (40, 300, 512 << 9), (128, 300, 512 << 9), (31, 300, 0)])
def test_line(k, P, line):
    for n, levels in ((1_000, 0 if line else 1), (line, 0), (line + 1, 1)):
        if not n:
            continue
        r, o = _reads(n, b"ACGT", k)
        got = gpu_count(r, o, k, P=P)
        assert kc.last_stats()["n_levels"] == levels, (n, kc.last_stats())
        assert_same(got, oracle.count(r, o, k), "%d bytes, k %d, P %d" % (n, k, P))


def test_options_split():
    r, o = _reads(100_000, b"ACGT", 1)
    for opts in (dict(shard_bits=8), dict(leaf_target=4000), dict(leaf_attempt=3000),
                 dict(table_slots_log2=11), dict(preagg=1), dict(mode=1)):
        gpu_count(r, o, 31, **opts)
        assert kc.last_stats()["n_levels"] >= 1, opts


@pytest.mark.parametrize("k", [21, 31, 40, 64, 100])
def test_overflowing_shard_is_split(k):
    r, o = _reads(262_000 if k <= 32 else 131_000, b"AT", 3)
    got = gpu_count(r, o, k, check=1)
    s = kc.last_stats()
    assert s["n_levels"] >= 1, s
    assert_same(got, oracle.count(r, o, k), "k %d" % k)
    assert s["valid_windows"] == int(got[1].sum())


@pytest.mark.parametrize("k", [21, 31, 64, 100])
def test_overflowing_shard_keeps_its_records(k):
    # the input is packed and its histogram taken once, as when it is split at once
    # (shard_bits = 8 gives the same shards)
    r, o = _reads(262_000 if k <= 32 else 131_000, b"AT", 3)
    best = {}
    for name, opts in (("after", dict(timing=1)), ("at once", dict(timing=1, shard_bits=8))):
        best[name] = 1e9
        for _ in range(15):
            gpu_count(r, o, k, **opts)
            t = kc.last_stats()["ms_stage"]
            best[name] = min(best[name], sum(t[s] for s in ("pack", "window_hist")))
    assert best["after"] < 1.5 * best["at once"], best
