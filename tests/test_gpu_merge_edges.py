"""Merging two results at the edges of the merge kernel's tiles: sizes just
below, at and above a tile, keys that both results hold on either side of a
tile's (and a thread's) boundary, and inputs that leave whole tiles to one side.
Against the merge oracle; integers, so every value must be equal."""
import numpy as np
import pytest

from oracle import post
import paper_2505_04431_amd as kc
from gpu_util import assert_same
from test_gpu_merge import _host, _torch_counts, _torch_keys

pytestmark = pytest.mark.gpu

TILE = {1: 2048, 2: 1024, 4: 512}


def _keys(ints, words):
    return post._words([x * 0x1_0000_0001 if words == 1 else (x << 60) + x // 3 for x in ints],
                       words)


@pytest.mark.parametrize("k,words", [(31, 1), (55, 2), (100, 4)])
@pytest.mark.parametrize("shape", ["one", "below", "at", "above", "pairs", "shifted", "apart",
                                   "sides", "rare"])
def test_merge_tile_edges(k, words, shape):
    t = TILE[words]
    every = list(range(3 * t))
    a, b = {
        "one": ([5], [5]),
        "below": (every[:t - 1:2], every[1:t - 1:2]),
        "at": (every[:t:2], every[1:t:2]),
        "above": (every[:t + 1:2], every[1:t + 1:2]),
        "pairs": (every, every),                  # every boundary falls between two pairs
        "shifted": (every, [0] + every[2:]),      # ... or inside one
        "apart": (every[:t + 7], every[t + 7:]),
        "sides": (every[t // 2:], every[:t + 3]),
        "rare": (every, every[::97]),
    }[shape]
    ac = np.arange(1, len(a) + 1, dtype=np.uint32)
    bc = np.arange(7, len(b) + 7, dtype=np.uint32)
    ak, bk = _keys(a, words), _keys(b, words)
    for x, xc, y, yc in ((ak, ac, bk, bc), (bk, bc, ak, ac)):
        got = kc.merge_counts(_torch_keys(x), _torch_counts(xc), _torch_keys(y),
                              _torch_counts(yc), k)
        assert_same(_host(*got), post.merge(x, xc, y, yc, words), shape)
