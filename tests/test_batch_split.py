"""The batched path where items are few (tiles split over several entries of
the tile list) and where they are many (more than a wave, more than the setup's
threads): every output against the float64 oracle."""

import numpy as np
import pytest

import workloads
from oracle import conv
from paper_1910_01972_amd import emu

TOL = 1e-5


def _items(n, seed):
    """Small uneven items, every 7th empty, of every batched FFT length."""
    g = np.random.Generator(np.random.PCG64(seed))
    out = []
    for i in range(n):
        N = int(2 ** g.integers(8, 13))
        Ns = 0 if i % 7 == 3 else int(g.integers(1, 6000))
        K, M = int(g.integers(1, 12)), int(g.integers(1, N // 2))
        s, h = workloads.make_signal_filters(Ns, K, M, seed=seed * 1000 + i)
        out.append((s, h, N))
    return out


def _check(items, outs):
    for (s, h, N), y in zip(items, outs):
        if len(s):
            want = conv.direct_conv(s, h)
            assert np.all(np.linalg.norm(y - want, axis=1) <= TOL * np.linalg.norm(want, axis=1)), (len(s), h.shape, N)


@pytest.mark.parametrize("n,grid", [(1, 64), (3, 16), (6, 200), (9, 5)])
def test_split_schedule_emulated(n, grid):
    items = _items(n, 70 + n)
    outs = emu.batched([{"s": s, "h": h, "N": N, "D": 0, "H": 0} for s, h, N in items], grid)
    _check(items, outs)


@pytest.mark.gpu
@pytest.mark.parametrize("n", [1, 5, 64, 65, 257, 600])
def test_item_counts(n):
    torch = pytest.importorskip("torch")
    from paper_1910_01972_amd import ols
    print(f"batch of {n} items", flush=True)
    items = _items(n, 300 + n)
    dev = [(torch.from_numpy(s).cuda(), torch.from_numpy(h).cuda(), N) for s, h, N in items]
    for make in (ols.OLSBatched, ols.OLSBatch):
        outs = [torch.full((h.shape[0], len(s)), complex(float("nan"), 0), dtype=torch.complex64, device="cuda")
                for s, h, _ in items]
        b = make(dev, outputs=outs)
        b.run()
        torch.cuda.synchronize()
        if make is ols.OLSBatched:
            assert b.status() == (0, -1)
        _check(items, [y.cpu().numpy() for y in outs])
