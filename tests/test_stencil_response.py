"""The transfer function that folded one-phase stencils multiply the segments'
spectra by, at every reach: rounded to float32 once (half a unit in the last
place of each component, beside what float64 leaves)."""

import numpy as np
import pytest

from paper_1910_01972_amd import emu

LENGTHS = (256, 512, 1024, 2048, 4096, 8192)


def rounded_once(got, want, scale):
    for g, w in ((got.real, want.real), (got.imag, want.imag)):
        assert np.all(np.abs(g.astype(np.float64) - w) <= 2.0 ** -24 * np.abs(w) + 1e-14 * scale)


@pytest.mark.parametrize("N", LENGTHS)
@pytest.mark.parametrize("T", [1, 2, 3, 4, 5, 8])
def test_transfer_function(N, T):
    rng = np.random.default_rng(N + T)
    k = np.arange(N)
    for left in range(T):
        w = rng.uniform(-1, 1, T).astype(np.float32)
        d = np.arange(T) - left
        phase = (k[:, None] * d) % N / N
        want = np.exp(2j * np.pi * phase) @ w.astype(np.float64)
        rounded_once(emu.stencil_response(N, w, left), want, np.abs(w).sum())
