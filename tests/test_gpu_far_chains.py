"""The far field by 16 groups of modes (eight waves of two chains, four of four),
against the FP64 oracle: numbers of modes around the groups, a wave's chains and a
tile of 256, in systems on both sides of the change from eight waves to four.

Tolerances: the library's bounds, 1e-12 (FP64) and 1e-5 (mixed) relative RMS."""
import numpy as np
import pytest

import oracle
import workloads
from test_gpu_parity import FP64_TOL, MIXED_TOL, Case, assert_close, dev  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("P", [2, 7, 11, 12, 13, 15, 16, 17, 24, 31, 33, 248, 255, 256, 257, 264, 271, 272, 273])
@pytest.mark.parametrize("N", [513, 32_767, 32_768])
def test_modes(dev, N, P, precision):  # noqa: F811
    """The first and last particles in cell order and 60 others."""
    w = workloads.Workload(f"chains_n{N}", N=N, kappa=0.5, gamma=1.0, r_c=2.5, P=P, seed=71)
    c = Case(dev, w, precision=precision)
    f, fn, _ = c.forces(6)
    n3, coef = c.ref.draw(6)
    rho = oracle.rho(c.st.x, c.st.q, w.L, n3)
    _, order = oracle.cells(c.st.x, w.L, w.r_c)
    idx = np.unique(np.concatenate([order[:66], order[-66:], workloads.rng(3, 1).integers(0, N, 60)]))
    fo = oracle.far_rb(c.st.x[:, idx], c.st.q[idx], w.L, n3, coef, rho)
    assert_close(f[:, idx] - fn[:, idx], fo, FP64_TOL if precision == 0 else MIXED_TOL, "far")
