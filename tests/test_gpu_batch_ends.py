"""Batch classes of several k: sets of a few reads, of lengths that leave a
class's last byte anywhere within a thread's window starts (the next set is of
another class, and its windows are not to be counted), the numbers of sets at
which a set id takes one bit more, set ids and k-mers of up to and more than 64
bits together, homopolymers. Against the oracle, bit-exact."""
import numpy as np
import pytest

import oracle
import paper_2505_04431_amd as kc
import synth
from gpu_util import assert_same, to_device

pytestmark = pytest.mark.gpu


def _sets(seed, n_sets, ks):
    rng = np.random.default_rng(seed)
    out = []
    for s in range(n_sets):
        k = ks[s % len(ks)]
        if s % 7 == 3:
            r = np.frombuffer([b"T", b"A", b"C"][s % 3] * 90 + b"ACGTN" * 4, dtype=np.uint8).copy()
            o = np.array([0, 40, 40, 41, r.size], dtype=np.uint64)
        else:
            g = synth.genome(seed * 1009 + s, int(rng.integers(120, 6000)))
            r, o = synth.reads(g, int(rng.integers(1, 200)), 100, err_rate=0.01, n_rate=0.001,
                               seed=seed + s)
        out.append((r, o, k))
    return out


@pytest.mark.parametrize("n_sets", [1, 2, 4, 5, 16, 17, 33, 130])
@pytest.mark.parametrize("shard_bits", [0, 1, 4, 5, 10])
def test_class_ends(n_sets, shard_bits):
    per_set = _sets(n_sets + 3, n_sets, [31, 32, 28, 30] if n_sets > 16 else [31, 32])
    reads = np.concatenate([r for r, _, _ in per_set])
    base = np.cumsum([0] + [r.size for r, _, _ in per_set])
    offs = np.concatenate([np.zeros(1, np.uint64)] +
                          [o[1:] + np.uint64(b) for (_, o, _), b in zip(per_set, base)])
    rt, ot = to_device(reads, offs)
    # a low leaf target, so that shards of a few thousand records are split
    for target in (0, 60):
        plan = kc.BatchPlan([o.size - 1 for _, o, _ in per_set], [r.size for r, _, _ in per_set],
                            [k for _, _, k in per_set], P=3,
                            opts=kc.options(shard_bits=shard_bits, leaf_target=target,
                                            leaf_attempt=target))
        keys, cnts, ends = plan.run(rt, ot)
        keys = keys.cpu().numpy().view(np.uint64)
        cnts = cnts.cpu().numpy().view(np.uint32)
        assert ends[-1] == keys.size
        for s, (r, o, k) in enumerate(per_set):
            a, b = int(ends[s]), int(ends[s + 1])
            assert_same((keys[a:b], cnts[a:b]), oracle.count(r, o, k),
                        "set %d of %d, k %d, leaf target %d" % (s, n_sets, k, target))
        plan.close()
