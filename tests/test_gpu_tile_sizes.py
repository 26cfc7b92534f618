"""Inputs that end exactly at, one below and one above a tile of the merge and of the
parser. Against their oracles, every value equal."""
import numpy as np
import pytest

from oracle import post
import paper_2505_04431_amd as kc
import synth
from gpu_util import assert_same
from test_gpu_merge import _host, _torch_counts, _torch_keys
from test_gpu_parse import _same

pytestmark = pytest.mark.gpu

# merged positions of a workgroup: 256 threads of 7, 5 and 3 positions (kMergeItems)
MERGE_TILE = {1: 256 * 7, 2: 256 * 5, 4: 256 * 3}
PARSE_TILE = 16384


def _keys(ints, words):
    return post._words([x * 0x1_0000_0001 if words == 1 else (x << 60) + x // 3 for x in ints],
                       words)


@pytest.mark.parametrize("k,words", [(31, 1), (55, 2), (100, 4)])
@pytest.mark.parametrize("tiles", [1, 2, 3])
@pytest.mark.parametrize("extra", [-2, -1, 0, 1, 2])
@pytest.mark.parametrize("shape", ["in turn", "apart", "one side", "pairs at the end",
                                   "pair over the end", "all pairs"])
def test_merge(k, words, tiles, extra, shape):
    n = tiles * MERGE_TILE[words] + extra  # na + nb
    every = list(range(n))
    a, b = {
        "in turn": (every[::2], every[1::2]),
        "apart": (every[:n // 3], every[n // 3:]),
        "one side": (every, []),
        # a key of both at the last two positions, or on either side of the tile's end
        "pairs at the end": (every[:n // 2], every[n // 2:n - 1] + [n + 5]),
        "pair over the end": (every[:-1], [n - 2]),
        "all pairs": (every[:n // 2], every[:n - n // 2]),
    }[shape]
    if shape == "pairs at the end":
        a = a[:-1] + [n + 5]
    assert len(a) + len(b) == n
    ac = np.arange(1, len(a) + 1, dtype=np.uint32)
    bc = np.arange(7, len(b) + 7, dtype=np.uint32)
    ak, bk = _keys(a, words), _keys(b, words)
    if not b:
        bk = ak[:0]
    for x, xc, y, yc in ((ak, ac, bk, bc), (bk, bc, ak, ac)):
        got = kc.merge_counts(_torch_keys(x), _torch_counts(xc), _torch_keys(y),
                              _torch_counts(yc), k)
        assert_same(_host(*got), post.merge(x, xc, y, yc, words), "%s, %d pairs" % (shape, n))


@pytest.mark.parametrize("fmt", ["fastq", "fasta"])
@pytest.mark.parametrize("tiles", [1, 2])
@pytest.mark.parametrize("extra", range(-3, 4))
@pytest.mark.parametrize("shift", [0, 5])
def test_parse(fmt, tiles, extra, shift):
    room = tiles * PARSE_TILE + extra - shift  # (the text starts `shift` into a tile)
    r, o = synth.ragged_reads(7, 1000, 20, 60)
    n = 1000
    make = synth.to_fastq if fmt == "fastq" else (lambda a, b: synth.to_fasta(a, b, width=0))
    while len(make(r, o[:n + 1])) > room - 40:
        n -= 1
    text = make(r, o[:n + 1])
    if fmt == "fastq":  # the last record's name makes up the length
        text += b"@" + b"x" * (room - len(text) - 9) + b"\nAC\n+\nII"
    else:
        text += b">" + b"x" * (room - len(text) - 5) + b"\nACG"
    assert len(text) == room
    _same(text, shift=shift)
