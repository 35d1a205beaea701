"""The cell build by its passes where their pieces can go wrong: cells of more
rows than a run holds, several runs of one cell in a wave and over many waves,
one tile of cells to thousands (more than a workgroup adds at once, more than the
last pass has threads), rows in random order and in the order of an earlier build
on another grid, and rows that moved in between; cell lists bit for bit the
oracle's stable sort."""
import numpy as np
import pytest

import oracle
import workloads
from test_gpu_parity import Case, dev  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
R = pytest.importorskip("paper_2501_10946_amd")


@pytest.mark.parametrize("clump", [0.0, 0.4, 1.0])
@pytest.mark.parametrize("N,r_c", [(4097, 2.0), (5000, 0.7), (20_000, 1.0), (70_001, 0.4), (300, 0.06)])
def test_cell_lists(dev, N, r_c, clump):  # noqa: F811
    w = workloads.Workload(f"passes_n{N}", N=N, kappa=1.0, gamma=1.0, r_c=r_c, P=3, seed=N, eps=0.1)
    st = workloads.clustered_state(w, clump, 0.9 * r_c)
    c = Case(dev, w, state=st, mmax=4)
    nc = int(np.floor(w.L / w.r_c))
    start = torch.full((nc ** 3 + 1,), -1, dtype=torch.int32, device=dev)
    order = torch.full((N,), -1, dtype=torch.int32, device=dev)
    g = workloads.rng(5, N)
    x = st.x
    for k in range(4):
        if k == 2:   # the next build starts from the order of the fine grid
            R.rbsog_rdf(c.sys.h, torch.tensor(x, device=dev), r_c, 4,
                        torch.zeros(4, dtype=torch.int64, device=dev))
        if k > 0:   # a tenth of the particles anywhere, the others a little away
            x = np.mod(x + 0.1 * r_c * g.standard_normal((3, N)), w.L)
            some = g.choice(N, N // 10, replace=False)
            x[:, some] = g.random((3, some.size)) * w.L
            x = np.ascontiguousarray(np.where(x >= w.L, 0.0, x))
        R.rbsog_build_cells(c.sys.h, torch.tensor(x, device=dev), start, order)
        want = oracle.cells(x, w.L, w.r_c)
        assert np.array_equal(start.cpu().numpy(), want[0])
        assert np.array_equal(order.cpu().numpy(), want[1])
