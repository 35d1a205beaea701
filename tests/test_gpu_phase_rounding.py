"""Rounding of the far field and of the structure factors against extended precision
(FP64): the errors stay below those of the forms that rotate a table entry by each phase,
then multiply by rho or by the charge, which were measured on these inputs (RMS error
over RMS value)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
import paper_2501_10946_amd as R  # noqa: E402

pytestmark = pytest.mark.gpu

LD = np.longdouble
PI = LD("3.14159265358979323846264338327950288")


def modes(h, step, P):
    n = torch.zeros((P, 3), dtype=torch.int32, device="cuda")
    coef = torch.zeros(P, dtype=torch.float64, device="cuda")
    R.rbsog_sample_k(h, step, n, coef)
    torch.cuda.synchronize()
    return n.cpu().numpy(), coef.cpu().numpy()


# eight particles around the sites of a lattice with no pair within the cutoff, so that
# the force is the far field alone; two charges; the table form's error
@pytest.mark.parametrize("kappa, edge, table_form", [(1.0, 3.01, 2.0348e-15), (0.5, 3.01, 2.2498e-15),
                                                     (0.5, 6.0, 3.1840e-15), (1.0, 12.0, 4.7701e-15)])
def test_far_force(orc, kappa, edge, table_form):
    r_c, N, P, evaluations = (2.0 if edge == 12.0 else 3.0), 8, 20, 400
    L = r_c * edge
    o = orc.sog_auto(1 / kappa, r_c, 1e-4)
    q = np.array([1.0, 2.0] * 4)
    s = R.System(q, np.ones(N), L, R.sog_from_parameters(o.lam, o.rc, o.h, o.t0, o.w, o.M1, o.M2), 1.0, P, seed=5,
                 device=torch.device("cuda"))
    rng = np.random.default_rng(11)
    site = np.stack(np.meshgrid([0.25, 0.75], [0.25, 0.75], [0.25, 0.75], indexing="ij")).reshape(3, 8)
    err = size = 0.0
    for step in range(evaluations):
        shift = rng.random((3, 1))
        x = np.mod(site + shift + 0.07 * (rng.random((3, N)) - 0.5), 1.0) * L
        x[x >= L] = 0
        xd = torch.tensor(x, device="cuda")
        f, f_near = torch.empty_like(xd), torch.empty_like(xd)
        R.rbsog_compute_forces(s.h, step, xd, f, f_near, None)
        n, coef = modes(s.h, step, P)
        assert float(f_near.abs().max()) == 0.0
        u = n.astype(LD) @ (x.astype(LD) / LD(L))
        th = 2 * PI * (u - np.rint(u))
        c, d = np.cos(th), np.sin(th)
        im = c * (q * d).sum(1)[:, None] - d * (q * c).sum(1)[:, None]
        exact = -(2 * PI / LD(L)) * q * ((coef.astype(LD)[:, None] * im).T @ n.astype(LD)).T
        err += float(((f.cpu().numpy() - exact) ** 2).sum())
        size += float((exact ** 2).sum())
    assert (err / size) ** 0.5 <= table_form


# equal charges in blobs of 256 consecutive particles (as cells hold them), long waves,
# an edge that is a power of two: what is left is the rounding of the terms and of their
# sums
def test_structure_factors_of_equal_charges(orc):
    N, P, L, table_form = 65536, 500, 16.0, 6.2498e-16
    o = orc.sog_auto(2.0, 4.0, 1e-4)
    q = np.ones(N)
    s = R.System(q, q, L, R.sog_from_parameters(o.lam, o.rc, o.h, o.t0, o.w, o.M1, o.M2), 1.0, P, seed=3,
                 device=torch.device("cuda"))
    rng = np.random.default_rng(7)
    err = size = 0.0
    for step in range(40):
        centre = np.repeat(rng.random((3, N // 256)), 256, axis=1)
        x = np.mod(centre + 0.1 * rng.random((3, N)), 1.0) * L
        x[x >= L] = 0
        rho = torch.zeros((P, 2), dtype=torch.float64, device="cuda")
        R.rbsog_compute_rho(s.h, step, torch.tensor(x, device="cuda"), rho)
        n, _ = modes(s.h, step, P)
        _, at = np.unique(n, axis=0, return_index=True)
        at = at[(n[at] ** 2).sum(1) <= 2]
        u = n[at].astype(LD) @ (x.astype(LD) / LD(L))
        th = 2 * PI * (u - np.rint(u))
        exact = np.stack([np.cos(th).sum(1), np.sin(th).sum(1)], 1)
        err += float(((rho.cpu().numpy()[at] - exact) ** 2).sum())
        size += float((exact ** 2).sum())
    assert (err / size) ** 0.5 <= table_form
