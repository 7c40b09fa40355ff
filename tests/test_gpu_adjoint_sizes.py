"""The adjoint on both sides of its size rules -- filters per unit at N = 4096,
and the launch that joins split windows and sums the dh slots (fewer values
than one of its workgroups holds, a ragged last chunk, several rounds of
chunks) -- against the float64 adjoint of eq. (1), relative L2 <= 1e-5 (per
filter row for dh)."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import workloads  # noqa: E402

pytestmark = pytest.mark.gpu
TOL = 1e-5

CASES = [  # N_s, K, M, N
    (300, 1, 3, 256), (5000, 3, 7, 512), (700, 2, 4, 1024), (300000, 5, 64, 1024), (400001, 4, 40, 2048),
    (9000, 1, 300, 4096), (40001, 16, 100, 4096), (200000, 16, 512, 4096), (120000, 31, 100, 4096),
    (500001, 31, 60, 4096), (60000, 3, 200, 8192),
]


@pytest.fixture(scope="module")
def loops():
    from oracle import loops as L
    if not L.available():
        L.build()
    return L


def rel(a, b):
    return np.linalg.norm(a - b, axis=-1) / np.linalg.norm(b, axis=-1)


@pytest.mark.parametrize("Ns,K,M,N", CASES)
def test_adjoint_size(loops, Ns, K, M, N):
    from paper_1910_01972_amd import ols
    print(f"adjoint size Ns={Ns} K={K} M={M} N={N}", flush=True)
    s, h = workloads.make_signal_filters(Ns, K, M, seed=N + K)
    g = workloads.make_grad(K, Ns, seed=N + K)
    plan = ols.OLSPlan(torch.from_numpy(h).cuda(), N=N)
    ts, tg = torch.from_numpy(s).cuda(), torch.from_numpy(g).cuda()
    nan = complex(float("nan"), float("nan"))
    ds = torch.full((Ns,), nan, dtype=torch.complex64, device="cuda")
    dh = torch.full((K, M), nan, dtype=torch.complex64, device="cuda")
    plan.backward(ts, tg, ds=ds, dh=dh)
    assert rel(ds.cpu().numpy(), loops.grad_signal(g, h)) <= TOL
    assert np.all(rel(dh.cpu().numpy(), loops.grad_filters(g, s, M)) <= TOL)
    # each gradient alone, and with the static scratch
    assert torch.equal(plan.backward(ts, tg, need_dh=False)[0], ds)
    assert torch.equal(plan.backward(ts, tg, need_ds=False)[1], dh)
    ds2, dh2 = plan.backward(ts, tg, static_scratch=True)
    assert rel(ds2.cpu().numpy(), ds.cpu().numpy()) <= 1e-6
    assert np.all(rel(dh2.cpu().numpy(), dh.cpu().numpy()) <= 1e-6)
    plan.close()
