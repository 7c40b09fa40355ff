"""ols_plan_get_call: what a forward call of a given size launches, against the
shape rule on the CPU, the tiling set, and the persistent grid."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import workloads  # noqa: E402
from paper_1910_01972_amd import emu  # noqa: E402

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("N,K,M,Ns,flags", [
    (256, 3, 20, 5000, ""), (512, 8, 32, 1 << 22, ""), (1024, 4, 64, 8192, ""), (1024, 8, 30, 300001, "real"),
    (1024, 128, 19, 40337, ""), (2048, 32, 256, 1 << 23, ""), (2048, 32, 256, 65536, ""), (2048, 32, 64, 1 << 22, ""),
    (2048, 24, 256, 262147, "real"), (2048, 32, 400, 741441, "power"), (4096, 16, 512, 1 << 18, ""),
    (4096, 32, 512, 1 << 23, ""), (4096, 4, 1300, 1290944, ""), (8192, 8, 2000, 1 << 18, ""), (8192, 3, 2000, 700001, "power"),
])
def test_call_is_what_the_rule_says(N, K, M, Ns, flags):
    from paper_1910_01972_amd import ols
    print(f"call report N={N} K={K} M={M} Ns={Ns} {flags}", flush=True)
    real, power = "real" in flags, "power" in flags
    make = workloads.make_real_signal_filters if real else workloads.make_signal_filters
    plan = ols.OLSPlan(dev(make(1, K, M, seed=1)[1]), N=N, power=power)
    cus, G, base = plan.launch()["cus"], N // 16, plan.launch()["block"]
    for nf in (0, 1, 2):
        if nf == 2 and N > (2048 if real else 4096):
            continue
        plan.set_tiling(nf, 0)
        full = plan.tiling()["max_workgroups_per_cu"] * cus
        for addr in (0, 8):
            if nf == 0 or addr == 0:
                y = None if addr == 0 else torch.empty(4, dtype=torch.float32, device="cuda")[addr // 4:]
                c = plan.call(Ns, y)
                want = emu.forward_shape(N, K, M, Ns, full=full, nf=nf, real=real, power=power, y_addr=addr)
                assert (c["filters_per_unit"], c["block"]) == want
                assert nf in (0, c["filters_per_unit"])
                segs = -(-Ns // c["hop"])
                trans = -(-segs // 2) if real else segs
                units = -(-trans // (c["block"] // G)) * -(-K // c["filters_per_unit"])
                assert c["grid"] == min(units, full * (base // c["block"]))
    plan.set_tiling(0, 1)
    assert plan.call(Ns)["grid"] <= cus * (base // plan.call(Ns)["block"])
    assert plan.call(0)["grid"] == 0
    with pytest.raises(ols.OLSError):
        plan.call(-1)
    plan.close()


@pytest.mark.parametrize("N,weights,folds", [(1024, [[-1.0, 1.0]], True), (4096, [[0.5, 0.5]], True),
                                             (2048, [[0.0, 1.0], [0.5, 0.5]], False)])
def test_tiling_of_a_stencil_is_reported_as_it_runs(N, weights, folds):
    """A folded stencil takes one filter per unit whatever tiling is asked for,
    and says so; a staged one takes the two it is given."""
    from paper_1910_01972_amd import ols
    print(f"stencil tiling report N={N}", flush=True)
    h = dev(workloads.make_signal_filters(1, 4, 30, seed=2)[1])
    plan = ols.OLSPlan(h, N=N, stencil=(weights, 1))
    plan.set_tiling(2, 0)  # accepted, as before
    want = 1 if folds else 2
    assert plan.tiling()["filters_per_unit"] == want and plan.call(100000)["filters_per_unit"] == want
    plan.close()
