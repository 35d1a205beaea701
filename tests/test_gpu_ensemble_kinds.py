"""The ensemble's shared launches: replicas of every kind of near field together
(FP64 by polynomials, FP64 by exponentials, mixed precision with one to twelve
Gaussians), one precision or one kind alone, more draws than a workgroup holds,
and enough workgroups for the partial sums to be spread through the launch; each
replica ends bit for bit as the same system stepped alone."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
R = pytest.importorskip("paper_2501_10946_amd")

DT = 0.01
POLY, EXP, MIXED = "poly", "exp", "mixed"
#       N, kappa, P, kind, steps
SETS = {
    "all kinds": [(500, 1.0, 40, POLY, 3), (900, 0.1, 257, EXP, 2), (700, 0.05, 300, MIXED, 3), (300, 2.0, 1, MIXED, 1),
                  (2000, 0.3, 100, EXP, 3)],
    "FP64 by exponentials": [(800, 0.5, 64, EXP, 2), (105, 1.0, 513, EXP, 3)],
    "FP64 by polynomials": [(800, 0.5, 256, POLY, 2)],
    "mixed precision": [(129, 0.02, 255, MIXED, 2), (800, 0.5, 64, MIXED, 3)],
    "partial sums spread, mixed precision": [(90_000, 1.0, 40, MIXED, 2), (130_000, 0.5, 30, MIXED, 2),
                                             (700, 1.0, 40, EXP, 2)],
    "partial sums spread, FP64": [(100_000, 1.0, 40, POLY, 2), (120_000, 1.0, 30, POLY, 1), (700, 1.0, 20, EXP, 2)],
}


@pytest.mark.parametrize("name", list(SETS))
def test_kinds(name, monkeypatch):
    dev = torch.device("cuda:0")
    ens = R.rbsog_ens_create(1 << 31, 8)
    try:
        reqs, slot_of = [], {}
        for i, (N, kappa, P, kind, steps) in enumerate(SETS[name]):
            w = workloads.Workload(f"k{i}", N=N, kappa=kappa, gamma=2.0, r_c=2.5, P=P, seed=70 + i)
            o = oracle.sog_auto(w.lam, w.r_c, w.eps)
            sog = R.sog_from_parameters(o.lam, o.rc, o.h, o.t0, o.w, o.M1, o.M2)
            prec = R.RBSOG_MIXED if kind == MIXED else R.RBSOG_FP64
            st = workloads.make_state(w)
            if kind == EXP:
                monkeypatch.setenv("RBSOG_NEAR_POLY", "0")
            else:
                monkeypatch.delenv("RBSOG_NEAR_POLY", raising=False)
            slot_of[R.rbsog_ens_admit(ens, R.make_params(N, w.L, w.kT, P, 9, i, 0, prec), sog, st.x, st.v, st.q, st.m,
                                      steps, DT)] = i
            s = R.System(st.q, st.m, w.L, sog, w.kT, P, seed=9, replica=i, precision=prec, device=dev)
            x, v = torch.tensor(st.x, device=dev), torch.tensor(st.v, device=dev)
            f, e = torch.empty_like(x), torch.zeros((steps, R.ENERGY_COLS), dtype=torch.float64, device=dev)
            R.rbsog_compute_forces(s.h, 0, x, f)
            R.rbsog_step(s.h, x, v, f, 0, steps, DT, e)
            R.rbsog_check(s.h)
            reqs.append((N, steps, x.cpu().numpy(), v.cpu().numpy(), e.cpu().numpy()))
        for _ in range(max(r[1] for r in reqs)):
            R.rbsog_ens_step(ens)
        torch.cuda.synchronize()
        done = R.rbsog_ens_poll(ens, 8)
        assert sorted(done) == sorted(slot_of)
        for slot in done:
            N, steps, xa, va, ea = reqs[slot_of[slot]]
            x, v, e = np.empty(3 * N), np.empty(3 * N), np.empty(R.ENERGY_COLS * steps)
            R.rbsog_ens_retire(ens, slot, x, v, e)
            assert np.array_equal(x.reshape(3, -1), xa)
            assert np.array_equal(v.reshape(3, -1), va)
            assert np.array_equal(e.reshape(-1, R.ENERGY_COLS), ea)
    finally:
        R.rbsog_ens_destroy(ens)
