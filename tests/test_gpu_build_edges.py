"""The cell build at the particle counts where its forms meet (one workgroup
with rows in registers, one workgroup through the snapshot, five launches):
cell lists bit for bit the oracle's stable sort, and two steps of a system at
rest on the oracle's trajectory.

Tolerances: none for the lists; 1e-12 for positions after two steps from rest
(displacements of ~1e-4 that differ by the forces' 1e-12 at most)."""
import numpy as np
import pytest

import oracle
import workloads
from test_gpu_parity import Case, dev  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
R = pytest.importorskip("paper_2501_10946_amd")


@pytest.mark.parametrize("clump", [False, True])
@pytest.mark.parametrize("N", [200, 1023, 1024, 1025, 2047, 4095, 4096, 4097])
def test_cell_lists(dev, N, clump):  # noqa: F811
    w = workloads.Workload(f"build_n{N}", N=N, kappa=1.0, gamma=1.0, r_c=2.0, P=3, seed=N)
    st = workloads.clustered_state(w, 0.3, 1.5) if clump else workloads.make_state(w)
    c = Case(dev, w, state=st)
    nc = int(np.floor(w.L / w.r_c))
    start = torch.full((nc ** 3 + 1,), -1, dtype=torch.int32, device=dev)
    order = torch.full((N,), -1, dtype=torch.int32, device=dev)
    want = oracle.cells(st.x, w.L, w.r_c)
    for _ in range(3):   # from the previous build's order
        R.rbsog_build_cells(c.sys.h, c.x, start, order)
        assert np.array_equal(start.cpu().numpy(), want[0])
        assert np.array_equal(order.cpu().numpy(), want[1])


@pytest.mark.parametrize("skin", [-1.0, 0.0])
@pytest.mark.parametrize("N", [1025, 4096, 4097, 16384, 16385])
def test_steps(dev, N, skin):  # noqa: F811
    """Velocities and masses move with their rows: unequal masses, each particle
    carrying its own force index through two builds."""
    w = workloads.Workload(f"build_n{N}", N=N, kappa=1.0, gamma=100.0, r_c=2.0, P=5, seed=N, dt=0.002)
    st = workloads.make_state(w)
    n = int(np.ceil(N ** (1 / 3)))
    site = workloads.rng(N, 5).permutation(n ** 3)[:N]
    x = (np.stack([site % n, site // n % n, site // n ** 2]) + 0.5) * (w.L / n)
    st = workloads.State(x=np.ascontiguousarray(x), v=np.zeros((3, N)), q=st.q,
                         m=workloads.rng(N, 4).uniform(0.5, 2.0, N))
    c = Case(dev, w, state=st, skin=skin)
    fo, _, _ = c.ref.force(st.x, 0)
    xo, vo = st.x.copy(), st.v.copy()
    x, v, f = c.x.clone(), torch.tensor(vo, device=dev), torch.tensor(fo, device=dev)
    R.rbsog_step(c.sys.h, x, v, f, 0, 2, w.dt)
    R.rbsog_check(c.sys.h)
    c.ref.run(xo, vo, fo, 0, 2, w.dt)
    assert np.abs(x.cpu().numpy() - xo).max() <= 1e-12
    assert np.abs(v.cpu().numpy() - vo).max() <= 1e-12 * max(1.0, np.abs(vo).max())
