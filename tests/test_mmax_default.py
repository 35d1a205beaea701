"""The default lattice cut-off of a system (the largest |n|^2 whose Fhat reaches
1e-16 of Fhat(0)) is the oracle's: with it given, the workspace, which holds the
lattice, has the same size, and one shell less or more changes it."""
import pytest

import oracle

R = pytest.importorskip("paper_2501_10946_amd")


@pytest.mark.parametrize("smooth", [1, 2])
@pytest.mark.parametrize("lam,r_c,eps", [(0.4, 2.0, 1e-3), (1.0, 3.0, 1e-4), (2.0, 4.0, 1e-5), (10.0, 5.0, 1e-4)])
@pytest.mark.parametrize("cells", [3.0, 3.7, 8.3, 20.0])
def test_mmax(lam, r_c, eps, smooth, cells):
    sog = R.rbsog_sog_init(lam, r_c, eps, smooth=smooth)
    L = r_c * cells
    o = oracle.sog_auto(lam, r_c, eps) if smooth == 1 else oracle.sog_auto2(lam, r_c, eps)
    mmax = oracle.mmax_default(o, L)

    def size(m):
        return R.rbsog_workspace_size(R.make_params(1000, L, 1.0, 10, 1, mmax=m), sog)

    assert size(0) == size(mmax)
    assert size(0) > size(max(1, mmax - 8)) and size(0) < size(mmax + 8)
