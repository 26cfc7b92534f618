"""Two-word keys on either side of the input size at which a plain call takes a
ninth shard bit, chosen by the library. Against the oracle, bit-exact."""
import pytest

import oracle
import synth
from gpu_util import assert_same, gpu_count

pytestmark = pytest.mark.gpu

LINE = 1920 << 16  # bytes: 256 leaves of the target in each of 256 shards


@pytest.mark.parametrize("k", [40, 64])
@pytest.mark.parametrize("n_reads", [LINE // 150 - 1, LINE // 150 + 2])
def test_about_the_line(k, n_reads):
    g = synth.genome(31, 6_000_000, [(3000, 40, 0.02)])
    r, o = synth.reads(g, n_reads, 150, err_rate=0.005, n_rate=0.0001, seed=9)
    assert_same(gpu_count(r, o, k, P=64, check=1), oracle.count(r, o, k),
                "%d reads, k %d" % (n_reads, k))
