"""The scratch that a table's buffer holds is what its arrays take, as the header states per element."""
import ctypes as C

import pytest

from test_abi import lib  # noqa: F401
from paper_1908_05936_amd import ct

FIXED = 256 + 16384 * 8 + 4096     # header, count partials, count words


def scratch(lib, chunk):  # noqa: F811
    d = ct.TableDesc(64, ct.VAL_U64, ct.HASH_MIX64, 8, chunk)
    nb = C.c_int64(0)
    assert lib.ct_table_bytes(C.byref(d), C.byref(nb)) == ct.CT_OK
    return nb.value - 8 * 128 - FIXED


@pytest.mark.parametrize("lg", range(10, 25))
def test_scratch_per_chunk_element(lib, lg):  # noqa: F811
    q = 1 << lg
    if q < 1 << 16:
        # repeated-key entries 2 x 8, mark 1, first copy 4, flag 1, slot 8; 4 per tile of 1024
        assert 0 <= scratch(lib, q) - 30 * q - 4 * (q // 1024) < 6 * 256
    else:
        # coarse bins (2 q / 512 + 256 in 512 segments) and fine bins (3 q), 12 bytes an entry, fill
        # counts, first occurrence 4, mark 1, first copy 4, flag 1, slot 8
        want = 12 * 512 * (2 * (q // 512) + 256) + 36 * q + 4 * (64 * 8 * 32 + q // 1024) + 18 * q + 4 * (q // 1024)
        assert 0 <= scratch(lib, q) - want < 12 * 256
        assert 78 <= scratch(lib, q) / q <= 104
