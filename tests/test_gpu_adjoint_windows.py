"""The adjoint's ds where one tile's filters are shared by several workgroups:
their partial windows are added four or eight at a time, so the counts at the
bounds of both, against the float64 adjoint of eq. (1), relative L2 <= 1e-5."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import workloads  # noqa: E402

pytestmark = pytest.mark.gpu
TOL = 1e-5


@pytest.fixture(scope="module")
def loops():
    from oracle import loops as L
    if not L.available():
        L.build()
    return L


# one tile, one unit per workgroup: as many windows as units (a filter each at
# N = 4096, two at N = 1024)
@pytest.mark.parametrize("N,Ns,per_unit", [(4096, 3000, 1), (1024, 3000, 2)])
@pytest.mark.parametrize("windows", [1, 2, 4, 5, 8, 9, 16, 17])
def test_windows(loops, N, Ns, per_unit, windows):
    from paper_1910_01972_amd import ols
    K, M = windows * per_unit, 40
    print(f"adjoint windows N={N} K={K}", flush=True)
    s, h = workloads.make_signal_filters(Ns, K, M, seed=K)
    g = workloads.make_grad(K, Ns, seed=K)
    plan = ols.OLSPlan(torch.from_numpy(h).cuda(), N=N)
    ds = torch.full((Ns,), complex(float("nan"), float("nan")), dtype=torch.complex64, device="cuda")
    plan.backward(torch.from_numpy(s).cuda(), torch.from_numpy(g).cuda(), need_dh=False, ds=ds)
    want = loops.grad_signal(g, h)
    assert np.linalg.norm(ds.cpu().numpy() - want) <= TOL * np.linalg.norm(want)
    plan.close()
