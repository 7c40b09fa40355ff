"""The delayed spectra: the phases they are multiplied by, rounded to float32
once, and how a bank's delays are shared out."""

import numpy as np
import pytest

from paper_1910_01972_amd import emu

LENGTHS = (256, 512, 1024, 2048, 4096, 8192)


def rounded_once(got, want, scale):
    for g, w in ((got.real, want.real), (got.imag, want.imag)):
        assert np.all(np.abs(g.astype(np.float64) - w) <= 2.0 ** -24 * np.abs(w) + 1e-14 * scale)


@pytest.mark.parametrize("N", LENGTHS)
def test_delay_phases(N):
    k = np.arange(N)
    for d in (1, 2, 5, 15, 16, 31):
        rounded_once(emu.delay_phases(N, d), np.exp(-2j * np.pi * ((k * d) % N / N)), 1.0)


def test_delay_rows():
    """Small banks spread the delays over the chip, large ones transform each
    filter once, and every delay has a row."""
    rows = emu.emu().ols_emu_delay_rows
    for blocks in (1, 4, 16, 31, 32, 33, 100, 250, 511, 512, 513, 5000):
        for delays in (16, 32):
            r = rows(blocks, delays, 256)
            assert 1 <= r <= delays and (r == delays or blocks * r >= 512) and blocks * (r - 1) < 512
