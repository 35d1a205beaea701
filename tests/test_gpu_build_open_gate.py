"""Builds of one workgroup with the gate open step after step, each from the order that
the one before left, against the passes: the same bits.  A system with the default skin
whose gate has been seen to be closed for a call takes the one workgroup in the next; the
same system with that skin given explicitly takes the passes."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
import paper_2501_10946_amd as R  # noqa: E402

pytestmark = pytest.mark.gpu

DT = 0.01


@pytest.mark.parametrize("N, langevin", [(4097, False), (10007, True), (16384, False)])
def test_same_bits_as_the_passes(orc, N, langevin):
    rng = np.random.default_rng(N)
    o = orc.sog_auto(2.0, 4.0, 1e-4)
    sog = R.sog_from_parameters(o.lam, o.rc, o.h, o.t0, o.w, o.M1, o.M2)
    L = (4 * np.pi * N / 3) ** (1 / 3)
    n = int(np.ceil(N ** (1 / 3)))
    site = rng.permutation(n ** 3)[:N]
    x0 = (np.stack([site % n, site // n % n, site // n ** 2]) + 0.5) / n * L
    q, m = rng.choice([1.0, 2.0], N), rng.choice([1.0, 3.0], N)
    slow = 1e-3 * rng.standard_normal((3, N))
    fast = 30.0 * rng.standard_normal((3, N))   # beyond half the skin (0.25) at every step
    states = []
    skin = -1.0
    for _ in range(2):
        s = R.System(q, m, L, sog, 1e-6, 40, seed=9, device=torch.device("cuda"), skin=skin)
        skin = s.info.skin
        assert skin > 0.0
        if langevin:
            R.rbsog_set_bath(s.h, R.RBSOG_BATH_LANGEVIN, 1.0, 1e-6)
        x, v = torch.tensor(x0, device="cuda"), torch.tensor(slow, device="cuda")
        f = torch.zeros_like(x)
        R.rbsog_step(s.h, x, v, f, 0, 30, 0.1 * DT)
        torch.cuda.synchronize()
        v.copy_(torch.tensor(fast))
        R.rbsog_step(s.h, x, v, f, 30, 20, DT)
        torch.cuda.synchronize()
        assert R.rbsog_get_info(s.h).skin == skin
        states.append((x, v, f))
    for a, b in zip(*states):
        assert torch.isfinite(a).all() and torch.equal(a, b)
