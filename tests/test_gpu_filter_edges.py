"""Spectrum and minimum-count filter at the edges of their tiles and loads: one
pair, sizes about a lane's four counts, a tile and many tiles, arrays that
start anywhere inside a larger one (the 16-byte loads need their alignment), and
keys of one, two and four words. Against the result-use oracles, bit-exact."""
import numpy as np
import pytest

from oracle import post
import paper_2505_04431_amd as kc
from gpu_util import assert_same
from test_gpu_merge import _host, _torch_counts, _torch_keys

pytestmark = pytest.mark.gpu


def _pairs(n, words, seed):
    rng = np.random.default_rng(seed)
    keys = rng.integers(0, 1 << 62, size=(n, words) if words > 1 else n, dtype=np.uint64)
    counts = np.where(rng.random(n) < 0.7, 1, rng.integers(1, 6000, size=n)).astype(np.uint32)
    return keys, counts


@pytest.mark.parametrize("k,words", [(31, 1), (55, 2), (100, 4)])
@pytest.mark.parametrize("n", [1, 3, 4, 5, 255, 1023, 4095, 4096, 4097, 8193, 40_003])
@pytest.mark.parametrize("skip", [0, 1, 2, 3])
def test_filter_edges(k, words, n, skip):
    keys, counts = _pairs(n + skip, words, n + skip)
    tk, tc = _torch_keys(keys)[skip:], _torch_counts(counts)[skip:]
    for least in (0, 1, 2, 3000, 6000):
        got = kc.filter_min_count(tk, tc, k, least)
        assert_same(_host(*got), post.filter_min_count(keys[skip:], counts[skip:], least),
                    "n %d from %d, at least %d" % (n, skip, least))


@pytest.mark.parametrize("n", [1, 3, 4, 5, 1023, 1024, 1025, 4099, 300_007])
@pytest.mark.parametrize("skip", [0, 1, 2, 3])
def test_spectrum_edges(n, skip):
    _, counts = _pairs(n + skip, 1, n)
    tc = _torch_counts(counts)[skip:]
    for most in (1, 2, 255, 4094, 4095, 4096, 5000, 200_000):
        assert np.array_equal(kc.spectrum(tc, most), post.spectrum(counts[skip:], most)), most


def test_spectrum_of_more_counts_than_the_grid_takes_at_once():
    n = 5_000_017
    rng = np.random.default_rng(1)
    counts = rng.integers(1, 50, size=n).astype(np.uint32)
    want = np.bincount(np.minimum(counts, 40), minlength=41)
    assert np.array_equal(kc.spectrum(_torch_counts(counts), 40), want.astype(np.uint64))
