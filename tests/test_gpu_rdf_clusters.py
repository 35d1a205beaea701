"""The pair histogram of clustered systems: the passes of crowded cell pairs are dealt to
many waves.  Counts against a plain count of all pairs (equal, but for pairs within 1e-9
of a bin's edge), and a bound on the time that one wave for all of a pair's particles
breaks (6000 of 20 000 particles in a sphere of 1.5: 109 ms so, 3 dealt out, 8.4 with a
thread per particle)."""
import time

import numpy as np
import pytest

torch = pytest.importorskip("torch")
import paper_2501_10946_amd as R  # noqa: E402

pytestmark = pytest.mark.gpu


def count(x, L, r_max, nbins):
    hist = torch.zeros(nbins, dtype=torch.int64, device="cuda")
    unsure = torch.zeros(nbins, dtype=torch.int64, device="cuda")
    N = x.shape[1]
    for a in range(0, N, 500):
        d = x[:, a:a + 500, None] - x[:, None, :]
        d -= L * torch.round(d / L)
        r = (d * d).sum(0).sqrt() / (r_max / nbins)
        r[torch.arange(r.shape[0]), torch.arange(a, a + r.shape[0])] = 2.0 * nbins
        r = r[r < nbins * (1 + 1e-12)]
        near = (r - r.round()).abs() < 1e-9
        b = r.floor().long().clamp(max=nbins - 1)
        hist += torch.bincount(b[~near], minlength=nbins)
        u = torch.bincount(r[near].round().long(), minlength=nbins + 1)
        unsure += u[:nbins] + u[1:]
    return hist, unsure


@pytest.mark.parametrize("N, clustered, radius, limit_ms", [
    (20000, 6000, 1.5, 20.0),    # a few cell pairs of ~600 particles
    (20000, 6000, 4.0, 8.0),
    (3000, 3000, 0.3, 8.0),      # all in one corner of the grid
    (5000, 0, 0.0, 8.0),
])
def test_histogram_of_clusters(N, clustered, radius, limit_ms):
    rng = np.random.default_rng(N + clustered)
    r_c, nbins = 4.0, 40
    L = (4 * np.pi * N / 3) ** (1 / 3)
    x = rng.random((3, N)) * L
    d = rng.standard_normal((3, clustered))
    d /= np.linalg.norm(d, axis=0)
    x[:, :clustered] = np.mod(0.1 + d * radius * rng.random(clustered) ** (1 / 3), L)   # across the faces
    x = torch.tensor(np.where(x >= L, 0.0, x), device="cuda")
    sog = R.rbsog_sog_init(2.0, r_c, 1e-4)
    s = R.System(np.ones(N), np.ones(N), L, sog, 1.0, 20, seed=3, device=torch.device("cuda"))
    hist = torch.zeros(nbins, dtype=torch.int64, device="cuda")
    times = []
    for _ in range(4):
        hist.zero_()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        R.rbsog_rdf(s.h, x, r_c, nbins, hist)
        torch.cuda.synchronize()
        times.append(1e3 * (time.perf_counter() - t0))
    want, unsure = count(x, L, r_c, nbins)
    off = hist - want
    assert bool((off >= 0).all()) and bool((off <= unsure).all())
    assert min(times) <= limit_ms
