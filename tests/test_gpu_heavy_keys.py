"""Inputs of few keys that occur very often: leaves of far more records than their
tables have slots, one key or several in them, alone and beside leaves of distinct
keys. Against the oracle, bit-exact."""
import numpy as np
import pytest

import oracle
from gpu_util import assert_same, gpu_count

pytestmark = pytest.mark.gpu


def _input(kind, n):
    rng = np.random.default_rng(11)
    rand = np.frombuffer(b"ACGT", dtype=np.uint8)[rng.integers(0, 4, n)].copy()
    if kind == "one key":
        r = np.full(n, ord("A"), dtype=np.uint8)
    elif kind == "few keys":
        r = np.resize(np.frombuffer(b"ACCGT", dtype=np.uint8), n).copy()
    elif kind == "errors":  # one key's copies with errors: a dense cluster beside it
        r = np.full(n, ord("A"), dtype=np.uint8)
        e = rng.random(n) < 0.002
        r[e] = rand[e]
    else:  # half of the reads random
        r = np.where((np.arange(n) // 151) % 2 == 0, np.uint8(ord("A")), rand)
    return r.astype(np.uint8), np.concatenate([np.arange(0, n, 151), [n]]).astype(np.uint64)


@pytest.mark.parametrize("k", [21, 32, 33, 63, 64, 65, 100, 128])
@pytest.mark.parametrize("kind", ["one key", "few keys", "errors", "half"])
@pytest.mark.parametrize("n", [300_000, 2_000_000])
def test_heavy_keys(k, kind, n):
    r, o = _input(kind, n)
    assert_same(gpu_count(r, o, k, P=3, check=1), oracle.count(r, o, k), "%s, k %d" % (kind, k))
