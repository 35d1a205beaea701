"""Structure factors by a launch of their own on both sides of the change to the
finer table of rotations (1536 workgroups), with one charge, one odd charge and
charges all different, whole groups of particles and a last one partly full;
FP64 against plain sums in extended precision at 40 of the modes.

Tolerance: the library's FP64 bound of 1e-12 of the RMS structure factor (the
phases, up to ~60 revolutions here, are good to ~2e-14 revolutions)."""
import math

import numpy as np
import pytest

import workloads
from test_gpu_rho_edges import reference

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
R = pytest.importorskip("paper_2501_10946_amd")


@pytest.mark.parametrize("charges", ["equal", "last", "all"])
@pytest.mark.parametrize("N,P", [(3000, 1024), (3001, 1050), (3067, 4096), (40_003, 257), (98_304, 256), (98_303, 255),
                                 (131_075, 300)])
def test_structure_factors(N, P, charges):
    dev = torch.device("cuda:0")
    w = workloads.Workload(f"fine_n{N}", N=N, kappa=0.5, gamma=1.0, r_c=2.5, P=P, seed=8)
    st = workloads.make_state(w)
    q = np.full(N, 1.7)
    if charges == "all":
        q = workloads.rng(N, 9).uniform(-1.0, 2.0, N)
    elif charges == "last":
        q[N - 1] = -0.6
    s = R.System(q, st.m, w.L, R.rbsog_sog_init(w.lam, w.r_c, w.eps), w.kT, P, seed=w.seed, device=dev)
    rho = torch.full((P, 2), 7.0, dtype=torch.float64, device=dev)
    R.rbsog_compute_rho(s.h, 3, torch.tensor(st.x, device=dev), rho)
    n = torch.zeros((P, 3), dtype=torch.int32, device=dev)
    R.rbsog_sample_k(s.h, 3, n, torch.zeros(P, dtype=torch.float64, device=dev))
    R.rbsog_check(s.h)
    at = np.unique(np.concatenate([[0, P - 1], workloads.rng(2, P).integers(0, P, 40)]))
    want = reference(st.x, q, w.L, n.cpu().numpy()[at])
    scale = max(math.sqrt(float((want ** 2).mean())), float(np.abs(q).max()))
    assert np.abs(rho.cpu().numpy()[at] - want).max() <= 1e-12 * scale
