"""The batched path where the work is small (equal shares of it, tiles cut between
workgroups), where it is dealt in whole tiles, and where items are many (more
than a wave, more than the setup's threads): every output against the float64
oracle."""

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


@pytest.mark.parametrize("n,grid", [(1, 64), (3, 16), (6, 200), (9, 5), (60, 1)])
def test_split_schedule_emulated(n, grid):
    items = _items(n, 70 + n)
    outs = emu.batched([{"s": s, "h": h, "N": N, "D": 0, "H": 0} for s, h, N in items], grid)
    _check(items, outs)


@pytest.mark.gpu
@pytest.mark.parametrize("log2_ns,K", [(19, 12), (22, 16)])
def test_shared_and_dealt(log2_ns, K):
    """Batches below and above the bound between shares and whole tiles, odd
    lengths, an empty item between: sampled outputs."""
    torch = pytest.importorskip("torch")
    from paper_1910_01972_amd import ols
    print(f"batch of 2^{log2_ns} x {K}", flush=True)
    shapes = [((1 << log2_ns) + 1, K, 40, 1024), (70001, 3, 300, 2048), (0, 2, 5, 256),
              ((1 << log2_ns) - 5, K, 500, 2048), (1 << log2_ns, K, 700, 4096)]
    items = [workloads.make_signal_filters(Ns, k, M, seed=40 + i) for i, (Ns, k, M, _) in enumerate(shapes)]
    outs = [torch.full((k, Ns), complex(float("nan"), 0), dtype=torch.complex64, device="cuda")
            for Ns, k, _, _ in shapes]
    b = ols.OLSBatch([(torch.from_numpy(s).cuda(), torch.from_numpy(h).cuda(), N)
                      for (s, h), (_, _, _, N) in zip(items, shapes)], outputs=outs)
    b.run()
    torch.cuda.synchronize()
    for (s, h), (Ns, k, M, N), y in zip(items, shapes, outs):
        if Ns == 0:
            continue
        assert not bool(torch.isnan(y.real).any())
        H = N - M
        idx = np.unique(np.clip((np.arange(0, Ns, max(1, Ns // 60 // H) * H)[:, None] + np.arange(-3, 4)).ravel(),
                                0, Ns - 1))
        want = conv.direct_conv_at(s, h, idx)
        got = y[:, torch.from_numpy(idx).cuda()].cpu().numpy()
        assert np.all(np.linalg.norm(got - want, axis=1) <= TOL * np.linalg.norm(want, axis=1)), (Ns, N)
    b.close()


@pytest.mark.gpu
@pytest.mark.parametrize("n", [1, 5, 64, 65, 256, 257, 600])
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
