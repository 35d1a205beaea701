"""The near field at the sizes where its work split can go wrong, against the
FP64 oracle: particle counts around a wave's 16 particles and a workgroup's 64,
particles with no neighbour beside particles with many, lists that overflow for
some particles of a wave and not for others, and cell pairs whose home particles
fill a list-build pass exactly, short of one or over by one.

Tolerance: the library's FP64 bound of 1e-12 relative to the oracle (a force is
a sum of at most ~100 terms here, each a few ulp off: below 1e-13)."""
import numpy as np
import pytest

import workloads
from test_gpu_parity import FP64_TOL, MIXED_TOL, Case, assert_close, assert_virials, dev  # noqa: F401

pytestmark = pytest.mark.gpu

L, R_C = 9.5, 3.0   # three coarse cells, six fine ones per axis


def case(dev, x, precision=0, skin=-1.0, edge=L):  # noqa: F811
    N = x.shape[1]

    class Boxed(workloads.Workload):
        L = edge   # this box, whatever the density

    w = Boxed(f"edges_n{N}", N=N, kappa=1.0, gamma=1.0, r_c=R_C, P=9, seed=40 + N)
    g = workloads.rng(90 + N, 2)
    st = workloads.State(x=np.ascontiguousarray(x), v=g.standard_normal((3, N)), q=g.uniform(0.5, 1.5, N),
                         m=np.ones(N))
    return Case(dev, w, state=st, precision=precision, skin=skin)


def check(c, precision=0):
    tol = FP64_TOL if precision == 0 else MIXED_TOL
    f, fn, e = c.forces(2)
    fo, fno, eo = c.ref.force(c.st.x, 2)
    if np.linalg.norm(fno) > 0:
        assert_close(fn, fno, tol, "near")
    else:
        assert np.abs(fn).max() == 0.0
    assert abs(e[0] - eo[0]) <= tol * abs(eo[0])
    assert_virials(e, eo, tol)


def uniform(n, seed):
    return workloads.rng(seed, 6).random((3, n)) * L


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("N", [1, 2, 15, 16, 17, 63, 64, 65, 257])
def test_particle_counts(dev, N, precision):  # noqa: F811
    check(case(dev, uniform(N, N), precision), precision)


@pytest.mark.parametrize("precision", [0, 1])
def test_empty_lists_beside_full_ones(dev, precision):  # noqa: F811
    """A clump of 20 particles and four particles out of reach of anything."""
    g = workloads.rng(7, 6)
    lone = np.array([[1.0, 6.5, 6.5, 1.0], [1.0, 1.0, 6.5, 6.5], [1.0, 6.5, 1.0, 6.5]])
    clump = np.array([[3.7], [3.7], [3.7]]) + 0.4 * g.random((3, 20))
    edge = 11.0
    c = case(dev, np.concatenate([lone, clump + 0.0], axis=1), precision, edge=edge)
    check(c, precision)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("cap", [8, 11])
def test_lists_that_overflow_for_some(dev, monkeypatch, cap, precision):  # noqa: F811
    """Capacities of 40 and 56 entries at about 45 neighbours within the list
    radius: both kinds of particle in most waves."""
    monkeypatch.setenv("RBSOG_NEAR_CAPACITY", str(cap))
    check(case(dev, uniform(300, 5), precision), precision)


@pytest.mark.parametrize("skin", [-1.0, 0.0])
@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 31, 32, 33])
def test_home_counts(dev, n, skin):  # noqa: F811
    """n particles in one cell, at the box corner and inside the box."""
    for corner in (0.05, 3.3):
        home = corner + 1.2 * workloads.rng(n, 8).random((3, n))
        check(case(dev, np.concatenate([home, uniform(70, 11)], axis=1), skin=skin))
