"""The numbers of leaves at which the launches change: all leaves to the
block-wide kernel up to 4,096, one workgroup for the output offsets up to
16,384. The bound the host has is 2 * bytes / leaf_target + 2 * 256 + 1, so the
leaf target moves it across both lines. Against the oracle, bit-exact."""
import numpy as np
import pytest

import oracle
import paper_2505_04431_amd as kc
import synth
from gpu_util import assert_same, gpu_count

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def reads():
    g = synth.genome(77, 20_000, [(900, 7, 0.02)])
    r, o = synth.reads(g, 799, 150, err_rate=0.01, n_rate=0.001, seed=3)
    # reads without a window, and a frequent k-mer, among them
    extra = np.frombuffer(b"A" * 400 + b"ACG" + b"N" * 40, dtype=np.uint8)
    ends = np.array([400, 403, 443], dtype=np.uint64)
    return np.concatenate([r, extra]), np.concatenate([o, o[-1] + ends])


@pytest.mark.parametrize("k", [4, 13, 31, 55])
@pytest.mark.parametrize("leaf_target", [14, 15, 16, 60, 66, 67, 68, 4000])
def test_leaf_numbers(reads, k, leaf_target):
    r, o = reads
    n = 2 * int(o[-1]) // leaf_target + 2 * 256 + 1
    assert n > 4096 or leaf_target > 60
    got = gpu_count(r, o, k, P=3, leaf_target=leaf_target, leaf_attempt=leaf_target, check=1)
    assert_same(got, oracle.count(r, o, k), "k %d, at most %d leaves" % (k, n))


@pytest.mark.parametrize("n", [1, 2, 150, 151, 3_000])
def test_few_reads(n):
    g = synth.genome(5, 5_000, [])
    r, o = synth.reads(g, n, 101, err_rate=0.01, seed=n)
    for k in (1, 21, 32, 40, 90):
        assert_same(gpu_count(r, o, k, P=2), oracle.count(r, o, k), "%d reads, k %d" % (n, k))


@pytest.mark.parametrize("k", [5, 21, 31, 55, 100])
@pytest.mark.parametrize("leaf_target", [930, 940, 945, 960, 3_000, 200_000])
def test_tiny_inputs(reads, k, leaf_target):
    """Up to 768 leaves of one-word keys are counted with the larger table at
    once; leaves of more distinct keys than that holds are refined."""
    r, o = reads
    want = oracle.count(r, o, k)
    for sb in (0, 1, 3):
        got = gpu_count(r, o, k, P=2, shard_bits=sb, leaf_target=leaf_target,
                        leaf_attempt=leaf_target, check=1)
        assert_same(got, want, "k %d, %d shard bits" % (k, sb))
        if sb == 1 and leaf_target == 200_000 and k == 31:
            assert kc.last_stats()["n_overflow"] > 0
