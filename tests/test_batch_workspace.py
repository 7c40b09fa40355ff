"""The workspace of a batched call keeps its size: programs that sized it once
(or hold a table of sizes) keep calling with it.  Host only, no GPU."""

import ctypes

import pytest

_lib = pytest.importorskip("paper_1910_01972_amd._lib")

# items -> bytes beside the filter spectra: a header, the twiddle tables, and
# 104 + 8 + 4 bytes per item, each part rounded up to 256 bytes
FIXED = {1: 64512, 2: 64512, 24: 66816, 64: 71424, 256: 93696, 257: 94208, 1000: 180224}


@pytest.mark.parametrize("n", sorted(FIXED))
def test_workspace_bytes(n):
    L, base = _lib.lib(), 1 << 40
    arr = (_lib.BatchItem * n)(*[_lib.BatchItem(base, 1000, base + (1 << 30), 3, 40, 1024, base + (2 << 30))] * n)
    out = ctypes.c_size_t()
    assert L.ols_batched_workspace_size(arr, n, ctypes.byref(out)) == 0
    assert out.value == FIXED[n] + n * 3 * 1024 * 8  # spectra K x N complex64
