"""Forward calls with banks that an XCD's L2 does not hold, and with re-aligned
rows of many filters, on both sides of the rules that choose their workgroups
(forward_shape): against the float64 oracle as the other call sizes, with the
shape that each is meant to run."""

import pytest

torch = pytest.importorskip("torch")

import test_gpu_call_sizes as sizes  # noqa: E402

pytestmark = pytest.mark.gpu

CASES = [  # N, K, M, N_s, flags, (filters per unit, threads)
    (1024, 1300, 60, 8000, "", (1, 256)), (1024, 1300, 60, 5040, "", (1, 64)), (1024, 2000, 60, 5041, "real", (1, 256)),
    (1024, 128, 19, 40337, "", (1, 256)), (1024, 1300, 19, 18241, "power", (1, 256)),
    (2048, 512, 400, 10001, "", (2, 256)), (2048, 512, 60, 10001, "", (1, 128)), (2048, 511, 400, 10001, "power", (2, 256)),
    (2048, 512, 400, 20001, "real", (2, 256)), (2048, 1024, 400, 23168, "", (1, 256)), (2048, 32, 400, 741441, "", (1, 256)),
    (2048, 600, 60, 111841, "real", (1, 256)), (4096, 4, 1300, 1290944, "", (2, 256)),
]


@pytest.mark.parametrize("N,K,M,Ns,flags,shape", CASES)
def test_large_bank(N, K, M, Ns, flags, shape):
    from paper_1910_01972_amd import ols
    import workloads
    make = workloads.make_real_signal_filters if "real" in flags else workloads.make_signal_filters
    plan = ols.OLSPlan(torch.from_numpy(make(16, K, M, seed=1)[1]).cuda(), N=N, power="power" in flags)
    ran = plan.call(Ns)
    plan.close()
    assert (ran["filters_per_unit"], ran["block"]) == shape
    sizes.test_call_size(N, K, M, Ns, flags)
