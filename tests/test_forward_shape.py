"""How a forward call runs -- filters per unit and threads per workgroup -- at
sizes on both sides of every rule, on a device of 256 CUs that holds two
workgroups of 256 threads (one of 512) per CU."""

import pytest

from paper_1910_01972_amd import emu

POWER, REAL, NO_DELAYS = dict(power=True), dict(real=True), dict(delays=False)

# N, K, M, N_s, what else, (filters per unit, threads)
CASES = [
    # N = 1024: one wave, unless the bank exceeds an XCD's L2 or many rows are off the grid
    (1024, 16, 200, 1482896, {}, (1, 64)), (1024, 256, 200, 92672, {}, (1, 64)),
    (1024, 512, 200, 10080, {}, (1, 256)), (1024, 512, 200, 2048, {}, (1, 64)),
    (1024, 1024, 19, 5040, {}, (1, 64)), (1024, 1024, 200, 5040, {}, (1, 256)),
    (1024, 1024, 19, 92672, {}, (1, 256)), (1024, 1300, 19, 18240, POWER, (1, 256)),
    (1024, 600, 19, 8592, REAL, (1, 64)), (1024, 600, 19, 39536, REAL, (1, 256)),
    (1024, 128, 19, 40336, {}, (1, 64)),
    (1024, 64, 19, 80673, {}, (1, 64)), (1024, 45, 19, 527249, {}, (1, 64)),
    (1024, 1433, 17, 16317, dict(power=True, delays=False, y_addr=32), (1, 256)),
    (1024, 1182, 133, 17888, dict(nf=2), (2, 256)), (1024, 16, 133, 17888, dict(nf=2), (2, 64)),
    # N = 2048: one filter per unit and one transform per workgroup, pairs where they give each one unit
    (2048, 32, 256, 1 << 18, {}, (1, 128)), (2048, 32, 256, 1 << 16, {}, (2, 128)), (2048, 32, 256, 1 << 23, {}, (1, 128)),
    (2048, 32, 256, 1 << 23, dict(nf=2), (2, 256)), (2048, 32, 256, 1 << 23, dict(nf=1), (1, 128)),
    # waves in step: short filters on the grid, long ones off it
    (2048, 32, 64, 1 << 22, {}, (1, 256)), (2048, 32, 64, 1 << 22, dict(y_addr=8), (1, 128)),
    (2048, 16, 64, 1 << 22, {}, (1, 128)), (2048, 32, 400, 741440, {}, (1, 128)),
    (2048, 16, 400, 5931633, {}, (1, 128)), (2048, 32, 64, 1 << 18, {}, (1, 128)),
    (2048, 32, 64, 100001, dict(full=128), (1, 128)), (2048, 32, 64, 100000, dict(full=128), (1, 256)),
    # large banks
    (2048, 600, 400, 39536, {}, (1, 128)), (2048, 600, 400, 39537, {}, (1, 256)),
    (2048, 1024, 400, 23168, {}, (1, 256)), (2048, 1300, 400, 18241, NO_DELAYS, (1, 256)),
    (2048, 1100, 200, 60001, NO_DELAYS, (1, 256)), (2048, 600, 60, 111840, POWER, (1, 256)),
    (2048, 600, 60, 111841, REAL, (1, 256)), (2048, 1024, 400, 5040, {}, (1, 128)),
    # N = 4096: pairs by what the longest workgroup gets
    (4096, 16, 512, 1 << 18, {}, (1, 256)), (4096, 32, 512, 1 << 23, {}, (2, 256)),
    (4096, 4, 1300, 1290944, {}, (2, 256)), (4096, 4, 60, 1290944, {}, (1, 256)), (4096, 4, 1571, 1710519, {}, (2, 256)),
    (4096, 7, 1300, 737680, {}, (1, 256)), (4096, 2, 1300, 2581888, POWER, (2, 256)), (4096, 2, 1300, 2581888, REAL, (1, 256)),
    # N = 8192 (one workgroup of 512 threads per CU), N = 512 and 256
    (8192, 2, 2048, 1 << 20, dict(full=256), (2, 512)), (8192, 8, 2048, 1 << 24, dict(full=256), (1, 512)),
    (512, 8, 32, 1 << 20, {}, (1, 64)), (512, 8, 32, 1 << 22, {}, (1, 256)), (256, 8, 20, 1 << 18, {}, (1, 64)),
]


@pytest.mark.parametrize("N,K,M,Ns,kw,want", CASES)
def test_forward_shape(N, K, M, Ns, kw, want):
    assert emu.forward_shape(N, K, M, Ns, **kw) == want
