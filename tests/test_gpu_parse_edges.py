"""FASTQ / FASTA parsing where its path changes: line ends past what the device
looks at, lines longer than a tile, texts that end about a tile's edge, every
number of lines before a tile's start, and outputs without room. Against the
parsing oracle, byte for byte."""
import ctypes

import numpy as np
import pytest

from oracle import fastx
import paper_2505_04431_amd as kc
import synth
from test_gpu_parse import _gpu_parse, _same, _text_tensor

pytestmark = pytest.mark.gpu

TILE = 16384


@pytest.mark.parametrize("fmt", ["fastq", "fasta"])
@pytest.mark.parametrize("before,after", [(0, 4096), (4095, 1), (4096, 0), (4097, 4097),
                                          (20_000, 0), (1, 50_000)])
def test_line_ends_around(fmt, before, after):
    r, o = synth.ragged_reads(5, 40, 0, 90, alphabet=b"ACGTN")
    text = (synth.to_fastq(r, o) if fmt == "fastq" else synth.to_fasta(r, o)).rstrip(b"\n")
    _same(b"\n" * before + text + b"\r\n" * after)


@pytest.mark.parametrize("n", [1, 4095, 4096, 4097, 40_000])
def test_nothing_but_line_ends(n):
    reads, offs, _ = kc.parse_fastx(_text_tensor(b"\n" * n))
    assert reads.numel() == 0 and offs.cpu().tolist() == [0]


@pytest.mark.parametrize("fmt", ["fastq", "fasta0", "fasta70"])
@pytest.mark.parametrize("crlf", [False, True])
def test_lines_longer_than_a_tile(fmt, crlf):
    r, o = synth.ragged_reads(6, 9, 10, 3 * TILE)
    text = synth.to_fastq(r, o, crlf=crlf) if fmt == "fastq" else \
        synth.to_fasta(r, o, width=int(fmt[5:]), crlf=crlf)
    for shift in (0, 3):
        _same(text, shift=shift)


@pytest.mark.parametrize("fmt", ["fastq", "fasta"])
@pytest.mark.parametrize("extra", range(-3, 4))
def test_text_about_a_tile(fmt, extra):
    # the last record is padded so that the text ends `extra` bytes from a tile's edge
    r, o = synth.ragged_reads(7, 160, 20, 60)
    make = synth.to_fastq if fmt == "fastq" else (lambda a, b: synth.to_fasta(a, b, width=0))
    for tiles in (1, 2):
        room = tiles * TILE + extra
        n = 160
        while len(make(r, o[:n + 1])) > room - 40:
            n -= 1
        text = make(r, o[:n + 1])
        pad = room - len(text)
        name = b"x" * (pad - (9 if fmt == "fastq" else 5) - (pad - 9) % 2 * (fmt == "fastq"))
        if fmt == "fastq":
            text += b"@" + name + b"\nAC\n+\nII\n"[:8]
        else:
            text += b">" + name + b"\nACG"
        _same(text.rstrip(b"\n"))


@pytest.mark.parametrize("lines", range(4))
def test_every_line_open_at_a_tile(lines):
    # the first record's name makes line `lines` the one open at the second tile
    name = b"n" * (TILE - 10 if lines == 0 else 5)
    seq = b"ACGT" * ((TILE if lines in (1, 2) else 8) // (4 if lines == 1 else 5))
    rec = b"@" + name + b"\n" + seq + b"\n+" + (b"p" * TILE if lines == 2 else b"") + b"\n"
    rec += b"I" * len(seq) + b"\n"
    more = b"@r\nACGTNACGT\n+\nIIIIIIIII\n" * 3000
    _same(rec * 2 + more)


def _parse_into(text, reads_room, records_room):
    import torch
    t = _text_tensor(text)
    reads = torch.full((max(1, reads_room),), 7, dtype=torch.uint8, device=t.device)
    offs = torch.full((records_room + 1,), 7, dtype=torch.int64, device=t.device)
    nr, nb = ctypes.c_uint64(9), ctypes.c_uint64(9)
    st = kc.lib().kc_parse_fastx(t.data_ptr(), t.numel(), 0, reads.data_ptr(), reads_room,
                                 offs.data_ptr(), records_room, ctypes.byref(nr),
                                 ctypes.byref(nb), None, None)
    return st, nr.value, nb.value, reads.cpu().numpy(), offs.cpu().numpy()


@pytest.mark.parametrize("fmt", ["fastq", "fasta"])
def test_outputs_without_room(fmt):
    r, o = synth.ragged_reads(8, 700, 20, 200)
    text = synth.to_fastq(r, o) if fmt == "fastq" else synth.to_fasta(r, o)
    n = int(o[-1])
    st, nr, nb, reads, offs = _parse_into(text, n, 700)
    assert (st, nr, nb) == (0, 700, n)
    assert np.array_equal(reads, r) and np.array_equal(offs.view(np.uint64), o)
    st, nr, nb, reads, offs = _parse_into(text, n - 1, 700)
    assert (st, nr, nb) == (-3, 700, n)
    assert (reads == 7).all() and (offs == 7).all()  # nothing written
    st, nr, nb, reads, offs = _parse_into(text, n, 699)
    assert (st, nr) == (-3, 700)
    assert (reads == 7).all() and (offs == 7).all()
    if fmt == "fastq":
        st, nr, nb, _, _ = _parse_into(text.replace(b"\n@r5 ", b"\n#r5 "), n, 700)
        assert (st, nr) == (-1, 0)
        st, nr, nb, _, _ = _parse_into(text.replace(b"\n@r5 ", b"\n#r5 "), n - 1, 700)
        assert (st, nr) == (-1, 0)
