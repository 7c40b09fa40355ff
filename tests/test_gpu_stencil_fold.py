"""One-phase stencils, applied to the segments' spectra up to N = 4096 and staged
above: every length, rows off the 128-byte grid (re-aligned rows leave room for
the stencil's reach), both reaches, the signal's ends, hops and tilings, against
the float64 oracle (relative L2 <= 1e-5 per row)."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import workloads  # noqa: E402
from oracle import post  # noqa: E402

pytestmark = pytest.mark.gpu
TOL = 1e-5
_W = np.random.default_rng(7).uniform(-1, 1, (1, 8)).astype(np.float32)
STENCILS = {"difference": ([[-1.0, 1.0]], 1), "behind": (_W.tolist(), 7), "ahead": (_W.tolist(), 0),
            "scale": ([[0.5]], 0)}


@pytest.mark.parametrize("Ns,K,M,N,name,flags", [
    (3001, 3, 20, 256, "behind", ""), (3001, 9, 20, 512, "ahead", "real"), (700, 2, 64, 1024, "difference", ""),
    (5000, 5, 64, 1024, "ahead", "real power"), (20001, 4, 300, 2048, "behind", "power"),
    (20001, 3, 300, 4096, "scale", ""), (30001, 2, 900, 8192, "ahead", ""),
    # rows re-aligned from 2^22 outputs per call on
    (530001, 8, 100, 1024, "ahead", ""), (530001, 8, 100, 2048, "behind", "power"), (530003, 8, 100, 2048, "ahead", "real"),
    (265001, 16, 500, 4096, "ahead", ""),
])
def test_one_phase_stencil(Ns, K, M, N, name, flags):
    from paper_1910_01972_amd import ols
    print(f"one-phase stencil Ns={Ns} K={K} M={M} N={N} {name} {flags}", flush=True)
    real, power = "real" in flags, "power" in flags
    w, left = STENCILS[name]
    make = workloads.make_real_signal_filters if real else workloads.make_signal_filters
    s, h = make(Ns, K, M, seed=N + K)
    plan = ols.OLSPlan(torch.from_numpy(h).cuda(), N=N, power=power, stencil=(w, left))
    dt = torch.float32 if real or power else torch.complex64
    y = torch.full((K, Ns), float("nan"), dtype=dt, device="cuda")
    ts = torch.from_numpy(s).cuda()
    plan.forward(ts, y)
    assert not bool(torch.isnan(y).any())
    H = plan.info()["H"]
    edges = np.concatenate([np.arange(0, Ns, max(1, Ns // 100 // H) * H), np.arange(Ns - 40, Ns, 8)])
    idx = np.unique(np.clip((edges[:, None] + np.arange(-9, 10)).ravel(), 0, Ns - 1))
    want = post.stencil_at(s, h, np.asarray(w, dtype=np.float32), left, idx, real=real)
    if power:
        want = np.abs(want) ** 2
    got = y[:, torch.from_numpy(idx).cuda()].cpu().numpy()
    assert np.all(np.linalg.norm(got - want, axis=1) <= TOL * np.linalg.norm(want, axis=1))
    # another hop and one workgroup per CU give the same rows to rounding
    plan.set_hop(max(1, H // 2))
    plan.set_tiling(0, 1)
    z = plan.forward(ts)
    assert bool((torch.linalg.vector_norm(z - y, dim=1) <= 2e-6 * torch.linalg.vector_norm(y, dim=1)).all())
    plan.close()
