"""Structure factors where the particle groups and the charges can go wrong:
counts around a group's size, groups left partly full, all charges equal (the
sums then run without them), all but one equal, the odd one in the first or last
place, and charges all different; FP64 against plain sums in extended precision.

Tolerance: the library's FP64 bound of 1e-12 of the RMS structure factor (the
phases, up to ~30 revolutions here, are good to ~1e-14 revolutions)."""
import math

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
R = pytest.importorskip("paper_2501_10946_amd")


def reference(x, q, L, n):
    u = (n.astype(np.longdouble) @ (x.astype(np.longdouble) / np.longdouble(L)))
    u = (u - np.rint(u)) * (2 * np.longdouble(math.pi) + np.longdouble(1.2246467991473532e-16) * 2)
    return np.stack([(q * np.cos(u)).sum(1), (q * np.sin(u)).sum(1)], 1).astype(np.float64)


@pytest.mark.parametrize("P", [1, 7, 64, 257])
@pytest.mark.parametrize("N", [1, 3, 7, 8, 9, 127, 128, 130, 515, 2049])
@pytest.mark.parametrize("charges", ["equal", "first", "last", "all"])
def test_structure_factors(N, P, charges):
    dev = torch.device("cuda:0")
    g = workloads.rng(1000 * N + P, 9)
    L = 11.0
    x = g.random((3, N)) * L
    q = np.full(N, 1.7)
    if charges == "all":
        q = g.uniform(-1.0, 2.0, N)
    elif charges != "equal":
        q[0 if charges == "first" else N - 1] = -0.6
    n = g.integers(-10, 11, (P, 3)).astype(np.int32)
    rho = torch.full((P, 2), 7.0, dtype=torch.float64, device=dev)
    R.rbsog_rho_noalloc(torch.tensor(x, device=dev), torch.tensor(q, device=dev), L, torch.tensor(n, device=dev), rho)
    want = reference(x, q, L, n)
    scale = max(math.sqrt(float((want ** 2).mean())), float(np.abs(q).max()))
    assert np.abs(rho.cpu().numpy() - want).max() <= 1e-12 * scale
