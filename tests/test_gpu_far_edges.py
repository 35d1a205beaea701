"""The far field where its tiles and its two layouts meet, against the FP64
oracle: numbers of modes around a wave's share and a tile of 256, and particle
counts on both sides of the change to two particles per lane, with the last
workgroup full, half empty and holding one particle.

Tolerances: the library's bounds, 1e-12 (FP64) and 1e-5 (mixed) relative RMS."""
import numpy as np
import pytest

import oracle
import workloads
from test_gpu_parity import FP64_TOL, MIXED_TOL, Case, assert_close, dev  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("P", [1, 3, 4, 5, 8, 9, 255, 256, 257, 265])
def test_mode_counts(dev, P, precision):  # noqa: F811
    w = workloads.Workload(f"modes_p{P}", N=321, kappa=1.0, gamma=1.0, r_c=2.0, P=P, seed=60 + P)
    c = Case(dev, w, precision=precision)
    f, fn, _ = c.forces(4)
    fo, fno, _ = c.ref.force(c.st.x, 4)
    assert_close(f - fn, fo - fno, FP64_TOL if precision == 0 else MIXED_TOL, "far")


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("N", [449_999, 450_000, 450_049, 450_113])
def test_two_particles_per_lane(dev, N, precision):  # noqa: F811
    """The last particles and 200 others of systems around the change of layout."""
    w = workloads.Workload(f"pair_n{N}", N=N, kappa=0.5, gamma=1.0, r_c=4.0, P=13, seed=70)
    c = Case(dev, w, precision=precision)
    f, fn, _ = c.forces(6)
    n3, coef = c.ref.draw(6)
    rho = oracle.rho(c.st.x, c.st.q, w.L, n3)
    _, order = oracle.cells(c.st.x, w.L, w.r_c)   # the last workgroups hold the last particles in cell order
    idx = np.unique(np.concatenate([order[-150:], workloads.rng(3, 1).integers(0, N, 200)]))
    fo = oracle.far_rb(c.st.x[:, idx], c.st.q[idx], w.L, n3, coef, rho)
    assert_close(f[:, idx] - fn[:, idx], fo, FP64_TOL if precision == 0 else MIXED_TOL, "far")
