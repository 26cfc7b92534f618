"""Texts that the parser refuses by their first byte: the outputs stay as they
were, whatever the number of lines and the room."""
import ctypes

import pytest

import paper_2505_04431_amd as kc
from test_gpu_parse import _text_tensor

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fmt", [kc.FASTX_AUTO, kc.FASTQ, kc.FASTA])
@pytest.mark.parametrize("records", [1, 4000])
@pytest.mark.parametrize("before", [0, 5000])
def test_first_byte_refused(fmt, records, before):
    import torch
    text = b"\n" * before + b"#r\nACGTACGT\n+\nIIIIIIII\n" + b"@r\nACGT\n+\nIIII\n" * (records - 1)
    t = _text_tensor(text)
    reads = torch.full((len(text),), 7, dtype=torch.uint8, device=t.device)
    offs = torch.full((records + 1,), 7, dtype=torch.int64, device=t.device)
    nr, nb = ctypes.c_uint64(9), ctypes.c_uint64(9)
    st = kc.lib().kc_parse_fastx(t.data_ptr(), t.numel(), fmt, reads.data_ptr(), len(text),
                                 offs.data_ptr(), records, ctypes.byref(nr), ctypes.byref(nb),
                                 None, None)
    assert (st, nr.value, nb.value) == (-1, 0, 0)
    if fmt == kc.FASTQ:
        assert b"line 0 " in kc.lib().kc_last_error()
    assert (reads == 7).all() and (offs == 7).all()
