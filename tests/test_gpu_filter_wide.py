"""The minimum-count filter of wider keys: kept pairs in every pattern about the
wave's and the tile's edges, against the filter oracle, every value equal; and its
time against its bytes (a key of W words costs no more than W words' share)."""
import time

import numpy as np
import pytest

from oracle import post
import paper_2505_04431_amd as kc
from gpu_util import assert_same
from test_gpu_merge import _host, _torch_counts, _torch_keys

pytestmark = pytest.mark.gpu

TILE, WAVE = 4096, 1024


@pytest.mark.parametrize("k,words", [(31, 1), (33, 2), (100, 4)])
@pytest.mark.parametrize("n", [1, 63, 65, WAVE - 1, WAVE + 1, TILE - 1, TILE, TILE + 1, 3 * TILE + 77])
@pytest.mark.parametrize("kept", ["all", "none", "first", "last", "every third", "runs"])
def test_kept_patterns(k, words, n, kept):
    i = np.arange(n)
    keep = {"all": i >= 0, "none": i < 0, "first": i % WAVE == 0, "last": i % WAVE == WAVE - 1,
            "every third": i % 3 == 0, "runs": (i // 61) % 2 == 0}[kept]
    counts = np.where(keep, 2 + i % 5, 1).astype(np.uint32)
    keys = post._words([int(x) * 0x1_0000_0001 if words == 1 else (int(x) << (64 * words - 40)) + int(x)
                        for x in i], words)
    got = kc.filter_min_count(_torch_keys(keys), _torch_counts(counts), k, 2)
    assert_same(_host(*got), (keys[keep], counts[keep]), "%d pairs, %s" % (n, kept))


def test_time_of_wider_keys():
    import ctypes

    import torch
    n, dev = 20_000_000, torch.device("cuda:0")
    counts = torch.randint(2, 50, (n,), dtype=torch.int32, device=dev)
    best = {}
    for k, words in ((31, 1), (55, 2), (100, 4)):
        keys = torch.zeros(n * words, dtype=torch.int64, device=dev)
        out_keys, out_counts = torch.empty_like(keys), torch.empty_like(counts)
        n_out = ctypes.c_uint64(0)
        best[words] = 1e9
        for _ in range(9):
            torch.cuda.synchronize()
            t = time.perf_counter()
            st = kc.lib().kc_filter_min_count(keys.data_ptr(), counts.data_ptr(), n, k, 2,
                                              out_keys.data_ptr(), out_counts.data_ptr(),
                                              ctypes.byref(n_out), None)
            best[words] = min(best[words], time.perf_counter() - t)
            assert st == 0 and n_out.value == n
    # bytes of a pair: 12, 20 and 36
    assert best[2] < best[1] * 20 / 12, best
    assert best[4] < best[1] * 36 / 12, best
