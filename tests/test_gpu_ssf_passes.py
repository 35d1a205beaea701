"""Static structure factors whose modes take one pass, one and a little, and
several passes of the structure-factor kernels, with the group size that makes
the passes few, and shells of fewer and more modes than a wave has lanes, against
the FP64 oracle.  Tolerance: the library's FP64 bound of 1e-12 of the largest
shell (the phases, up to ~15 revolutions, are good to ~1e-14 revolutions)."""
import math

import numpy as np
import pytest

import oracle
import workloads
from test_gpu_observables import dev, gpu_ssf  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,m_s", [(700, 1), (700, 39), (3000, 40), (3000, 62), (2999, 90), (9000, 63)])
def test_passes(dev, N, m_s):  # noqa: F811
    L = (4 * math.pi * N / 3) ** (1 / 3)
    st = workloads.small_system(N, L, seed=N + m_s)
    s = gpu_ssf(dev, st.x, st.q, L, m_s)
    so = oracle.ssf(st.x, st.q, L, m_s)
    assert np.all(s[so == 0] == 0.0)
    assert np.abs(s - so).max() <= 1e-12 * np.abs(so).max()
