"""Energy histories around the number of rows one launch adds (16): the rows of a
run are bit for bit those of the same run in calls of one step (plain
trajectories and the full lattice, which has one row per launch), and the first
rows of a longer run (also with a global bath, whose rows report the kinetic
energy after its closing half-step; a bath's run in several calls rounds its
velocity factors one by one instead of their product, so its bits differ)."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
R = pytest.importorskip("paper_2501_10946_amd")


def rows(kind, calls):
    dev = torch.device("cuda:0")
    w = workloads.Workload("rows", N=600, kappa=1.0, gamma=1.0, r_c=2.5, P=20, seed=9)
    st = workloads.make_state(w)
    sog = R.rbsog_sog_init(w.lam, w.r_c, w.eps)
    s = R.System(st.q, st.m, w.L, sog, w.kT, w.P, seed=w.seed, mmax=12, full_k=kind == "full lattice", device=dev)
    if kind == "nose-hoover":
        R.rbsog_set_bath(s.h, R.RBSOG_BATH_NOSE_HOOVER, 2.0, w.kT)
    x, v = torch.tensor(st.x, device=dev), torch.tensor(st.v, device=dev)
    f = torch.empty_like(x)
    R.rbsog_compute_forces(s.h, 0, x, f)
    e = torch.full((sum(calls) + 1, R.ENERGY_COLS), -7.0, dtype=torch.float64, device=dev)
    at = 0
    for n in calls:
        R.rbsog_step(s.h, x, v, f, at, n, w.dt, e[at:])
        at += n
    R.rbsog_check(s.h)
    e = e.cpu().numpy()
    assert np.all(e[-1] == -7.0) and np.all(e[:-1, 5] > 0.0)
    return e[:-1]


@pytest.mark.parametrize("kind", ["plain", "nose-hoover", "full lattice"])
@pytest.mark.parametrize("nsteps", [1, 15, 16, 17, 33])
def test_rows(nsteps, kind):
    e = rows(kind, [nsteps])
    assert np.array_equal(e, rows(kind, [nsteps + 20])[:nsteps])
    if kind != "nose-hoover":
        assert np.array_equal(e, rows(kind, [1] * nsteps))
