"""The order of a near launch's structure-factor workgroups (before the near ones or
spread among them) changes no bit: forces, near forces and energies on both sides of
the lines between the two orders, by the library's choice and with either forced."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
R = pytest.importorskip("paper_2501_10946_amd")


@pytest.mark.parametrize("precision,N,P", [(0, 284_160, 500), (0, 284_161, 500), (0, 7, 500), (1, 96_000, 500),
                                           (1, 102_000, 500), (1, 200_003, 7)])
def test_orders(precision, N, P, monkeypatch):
    dev = torch.device("cuda:0")
    w = workloads.Workload(f"spread_n{N}", N=N, kappa=0.5, gamma=1.0, r_c=min(2.5, 0.5 * N ** (1 / 3)), P=P, seed=3)
    st = workloads.make_state(w)
    s = R.System(st.q, st.m, w.L, R.rbsog_sog_init(w.lam, w.r_c, w.eps), w.kT, P, seed=3, precision=precision,
                 device=dev)
    x = torch.tensor(st.x, device=dev)
    out = []
    for order in (None, "0", "1"):
        if order is None:
            monkeypatch.delenv("RBSOG_NEAR_INTERLEAVE", raising=False)
        else:
            monkeypatch.setenv("RBSOG_NEAR_INTERLEAVE", order)
        f, fn = torch.full_like(x, 7.0), torch.full_like(x, 7.0)
        e = torch.full((R.ENERGY_COLS,), 7.0, dtype=torch.float64, device=dev)
        R.rbsog_compute_forces(s.h, 2, x, f, fn, e)
        R.rbsog_check(s.h)
        out.append([a.cpu().numpy() for a in (f, fn, e)])
    for other in out[1:]:
        for a, b in zip(out[0], other):
            assert np.array_equal(a, b) and np.all(np.isfinite(a))
