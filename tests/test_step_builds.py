"""The cell build that a system's steps take (host only, no GPU).  One workgroup builds
up to 4096 particles whatever the gate does, and up to 16 384 only once the gate has
been seen to be open in at most one of N / 1024 steps; a system that has not been looked at,
that rebuilds more often, or whose rebuilds are not counted takes the passes."""
import subprocess

import pytest

from host_runtime import program

ONE, PASSES = (20, 0), (0, 20)


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    return program("step_builds_check", tmp_path_factory.mktemp("builds"))


@pytest.mark.parametrize("N, every, skin, calls", [
    (4096, 1, -1.0, [ONE] * 4),                    # small: rows in registers
    (4096, 1, 0.5, [ONE] * 4),
    (4097, 0, -1.0, [PASSES, ONE, ONE, ONE]),      # looked at after the first call
    (16384, 20, -1.0, [PASSES, ONE, ONE, ONE]),
    (16384, 10, -1.0, [PASSES] * 4),               # two of 20 steps
    (10007, 10, -1.0, [PASSES, ONE, ONE, ONE]),
    (10007, 5, -1.0, [PASSES] * 4),
    (4200, 5, -1.0, [PASSES, ONE, ONE, ONE]),
    (4200, 2, -1.0, [PASSES] * 4),
    (16384, 0, 0.5, [PASSES] * 4),                 # an explicit skin: not counted
    (8000, 1, 0.5, [PASSES] * 4),
    (16385, 0, -1.0, [PASSES] * 4),                # more rows than it holds
])
def test_build_of_steps(exe, N, every, skin, calls):
    r = subprocess.run([exe, str(N), str(every), str(skin)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
    assert [tuple(map(int, line.split())) for line in r.stdout.splitlines()] == calls
