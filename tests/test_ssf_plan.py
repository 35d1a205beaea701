"""The passes of rbsog_ssf (host only, no GPU): whatever the last pass is left
with, every launch of partial sums stays within the staging area and the
scratch, and no call is refused.  Sizes whose last pass is short: 76 modes of
4 082 034 at N = 50 000, m_s = 9 829, and 75 of 4 096 290 at N = 60 000, m_s =
9 851; beside them the smallest calls, calls of one pass and of a few, and a large one."""
import subprocess

import pytest

from host_runtime import program


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    return program("ssf_passes_check", tmp_path_factory.mktemp("ssf"))


@pytest.mark.parametrize("calls", [
    [(1, 1), (1, 40), (7, 100), (300, 90), (1000, 41), (2000, 300)],
    [(20000, 10), (20000, 100), (65536, 100), (100000, 64), (1000000, 100)],
    [(50000, 9829)],
    [(60000, 9851)],
])
def test_every_pass_is_in_bounds(exe, calls):
    args = [str(v) for c in calls for v in c]
    r = subprocess.run([exe, *args], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "0 failures" in r.stdout
