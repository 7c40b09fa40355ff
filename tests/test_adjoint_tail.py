"""The adjoint's tail on the CPU: which dh slots it reads against which the
adjoint kernels write (all three kinds of unit), which tiles it finishes, how
its work is cut, and the emulated adjoint, whose scratch starts as NaN, at
grids that leave workgroups less than a tile."""

import numpy as np
import pytest

import workloads
from oracle import adjoint
from paper_1910_01972_amd import emu


def owned(U, P, b):
    return range(U * b // P, U * (b + 1) // P)


@pytest.mark.parametrize("segs,paired,fpu", [(1, False, 1), (1, False, 2), (2, True, 2), (4, True, 2), (8, True, 2),
                                             (16, True, 2)])
def test_slots_read_are_slots_written(segs, paired, fpu):
    rng = np.random.default_rng(segs + 100 * fpu)
    for _ in range(60):
        K, ntiles = int(rng.integers(1, 20)), int(rng.integers(1, 12))
        upt = -(-K // fpu)
        U = ntiles * upt
        P = int(rng.integers(1, U + 1))
        want = np.zeros((P * segs, K), dtype=bool)
        for b in range(P):
            for u in owned(U, P, b):
                for r in range(fpu * (u % upt), min(K, fpu * (u % upt) + fpu)):
                    for grp in range(segs):
                        if not paired or (grp & 1) == (r & 1):
                            want[b * segs + grp, r] = True
        assert np.array_equal(emu.dh_slots(U, P, upt, fpu, segs, paired, K), want), (K, ntiles, P)


@pytest.mark.parametrize("by_tile", [False, True])
def test_split_tiles_are_finished_once(by_tile):
    rng = np.random.default_rng(5)
    for _ in range(200):
        upt, ntiles = int(rng.integers(1, 30)), int(rng.integers(1, 30))
        U = upt * ntiles
        P = int(rng.integers(1, U + 1))
        owner = {u: b for b in range(P) for u in owned(U, P, b)}
        want = [(t, owner[t * upt], owner[(t + 1) * upt - 1]) for t in range(ntiles)]
        want = [w for w in want if w[1] != w[2]]
        got = [emu.split_tile(U, P, upt, by_tile, i) for i in range(ntiles if by_tile else P - 1)]
        assert sorted(g for g in got if g) == want, (upt, ntiles, P)


def test_tail_shape_bounds_what_a_lane_waits_for():
    """(segs, H, tiles, units per tile, grid, K M): few tiles of many workgroups,
    many segments per tile, many slots of few lags, the ordinary sizes between,
    and calls without a split tile."""
    for segs, H, ntiles, upt, grid, KM in [
            (1, 4080, 2, 59, 118, 59), (2, 1344, 5, 40, 200, 79 * 691), (16, 240, 750, 3, 512, 18),
            (16, 240, 32, 4, 128, 24), (8, 256, 23, 6, 138, 2816), (4, 960, 13, 2, 26, 256), (1, 3584, 1171, 8, 512, 8192),
            (1, 6144, 300, 16, 256, 4096), (16, 240, 680, 1, 512, 12), (16, 1, 9, 1, 9, 1), (1, 4000, 1, 1, 1, 5),
            (4, 960, 1024, 7, 512, 256)]:
        t = emu.tail_shape(segs, H, ntiles, upt, grid, KM)
        U = ntiles * upt
        split = any((U * b // grid) % upt for b in range(1, grid))
        assert bool(t["nfix"]) == split
        if split:
            assert t["nfix"] == min(ntiles, grid - 1) and t["by_tile"] == (ntiles < grid - 1)
            lanes = 256 * t["split"]
            assert (t["split"] - 1) * 256 < segs * H  # no workgroup without an output
            assert -(-segs * H // lanes) <= 4 and (t["nfix"] > 64 or lanes >= segs * H)
        assert t["ndh"] % 8 == 0 and t["ndh"] * t["lags"] >= KM > (t["ndh"] - 8) * t["lags"]
        rounds = -(-(-(-grid * segs // 16)) // (256 // t["lags"]))
        assert rounds <= 4 or KM // t["lags"] >= 512


@pytest.mark.parametrize("N,Ns,K,M,grid", [(256, 9000, 5, 30, 1000), (256, 9000, 5, 30, 3), (1024, 7000, 7, 100, 9),
                                           (2048, 6000, 11, 300, 20), (4096, 9000, 3, 700, 8), (8192, 9000, 2, 50, 3)])
def test_emulated_adjoint_reads_what_was_written(N, Ns, K, M, grid):
    s, h = workloads.make_signal_filters(Ns, K, M, seed=N + K)
    gy = workloads.make_grad(K, Ns, seed=N + K)
    D = -(-(M - 1) // 16) * 16
    ds, dh, guards = emu.backward(s, gy, h, N, D, N - D, grid)
    assert guards
    for got, want in ((ds, adjoint.grad_signal(gy, h)), (dh, adjoint.grad_filters(gy, s, M))):
        assert np.all(np.linalg.norm(got - want, axis=-1) <= 1e-5 * np.linalg.norm(want, axis=-1))
