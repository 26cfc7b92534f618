"""Leaves of keys of two and four words, at the sizes where their path changes:
leaves that just fit a table, that overflow it into the second count's, and that
overflow that as well; clusters of keys with a long common prefix (ranked in
large groups, or sorted), and one key many times over. Bit-exact."""
import numpy as np
import pytest

import oracle
import paper_2505_04431_amd as kc
import synth
from gpu_util import assert_same, gpu_count

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def inputs():
    # mostly distinct windows
    spread = synth.ragged_reads(3, 500, 100, 400)
    # copies of one read that differ near their ends: keys alike in their first bases
    rng = np.random.default_rng(8)
    base = np.frombuffer(b"ACGT", dtype=np.uint8)
    one = base[rng.integers(0, 4, 140)]
    rows = np.tile(one, (900, 1))
    at = rng.integers(70, 140, size=(900, 3))
    rows[np.arange(900)[:, None], at] = base[rng.integers(0, 4, (900, 3))]
    cluster = rows.reshape(-1), np.arange(901, dtype=np.uint64) * np.uint64(140)
    # one key, and its neighbours, thousands of times
    same = np.tile(one, 400), np.arange(401, dtype=np.uint64) * np.uint64(140)
    return {"spread": spread, "cluster": cluster, "same": same}


@pytest.mark.parametrize("k", [33, 63, 64, 65, 100, 128])
@pytest.mark.parametrize("kind", ["spread", "cluster", "same"])
@pytest.mark.parametrize("leaf_target", [0, 1790, 1800, 3600, 100_000])
def test_wide_leaves(inputs, k, kind, leaf_target):
    r, o = inputs[kind]
    # one shard bit: leaves as large as the target allows
    got = gpu_count(r, o, k, P=1, shard_bits=1, leaf_target=leaf_target, leaf_attempt=leaf_target,
                    check=1, timing=1)
    st = kc.last_stats()
    assert_same(got, oracle.count(r, o, k), "%s, k %d, leaf target %d" % (kind, k, leaf_target))
    if kind == "spread" and leaf_target == 3600:
        assert st["second_records"] > 0  # distinct keys past one table, within two
    if kind == "spread" and leaf_target == 100_000:
        assert st["n_overflow"] > 0      # past both
