"""The FASTA reader's functions start on cache lines, wherever the rest of the
library ends: its byte loops lose up to a fifth of their speed elsewhere."""
import ctypes

import pytest

from paper_2509_13300_amd import _lib as L


@pytest.mark.parametrize("name", ["ah_fasta_count", "ah_fasta_read"])
def test_reader_starts_on_a_cache_line(name):
    # the library is mapped at a page, so an address's low bits are the file's
    assert ctypes.cast(getattr(L.lib(), name), ctypes.c_void_p).value % 64 == 0
