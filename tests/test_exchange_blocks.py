"""The exchanges of a transform that spans several waves leave out every barrier
that only guards a wave's own block of LDS cells."""

import pytest

from paper_1910_01972_amd import emu


@pytest.mark.parametrize("N", [2048, 4096, 8192])
def test_waves_keep_to_their_blocks(N):
    # 1024 positions and their padding: at least 1024 cells, the same in both layouts
    assert emu.wave_block(N) >= 1024
