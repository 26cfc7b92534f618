"""Texts with very many line ends before and after their records, about the distance
up to which the device looks for the first and last byte itself. Against the parsing
oracle, byte for byte."""
import pytest

import paper_2505_04431_amd as kc
import synth
from test_gpu_parse import _same, _text_tensor

pytestmark = pytest.mark.gpu

MOST = 1 << 20  # bytes that the device looks at from either end
STEP = 4096


@pytest.mark.parametrize("fmt", ["fastq", "fasta"])
@pytest.mark.parametrize("before,after", [
    (STEP - 1, STEP), (STEP, STEP - 1), (2 * STEP + 1, 3 * STEP), (MOST - 1, 0), (MOST, 0),
    (MOST + 1, 0), (0, MOST - 1), (0, MOST), (0, MOST + 1), (MOST + 1, MOST + 1), (MOST + 1, 5),
    (7, 2 * MOST + 3)])
def test_line_ends(fmt, before, after):
    r, o = synth.ragged_reads(5, 40, 0, 90, alphabet=b"ACGTN")
    text = (synth.to_fastq(r, o) if fmt == "fastq" else synth.to_fasta(r, o)).rstrip(b"\n")
    _same(b"\n" * before + text + b"\n" * after)
    _same(b"\r\n" * (before // 2) + text + b"\r\n" * (after // 2), shift=3)


@pytest.mark.parametrize("n", [STEP + 1, MOST - 1, MOST, MOST + 1, 2 * MOST + 5])
def test_nothing_but_line_ends(n):
    reads, offs, _ = kc.parse_fastx(_text_tensor(b"\n" * n))
    assert reads.numel() == 0 and offs.cpu().tolist() == [0]


@pytest.mark.parametrize("before", [0, MOST - 1, MOST, MOST + 9])
def test_one_byte(before):
    _same(b"\n" * before + b">")
    _same(b">" + b"\n" * before)
