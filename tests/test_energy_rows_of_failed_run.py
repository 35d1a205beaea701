"""The energy rows of a run that fails at a launch (host only, no GPU): every step that
was enqueued whole has its row, whichever launch fails, though rows are added sixteen at
a time."""
import subprocess

import pytest

from host_runtime import program


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    return program("energy_rows_check", tmp_path_factory.mktemp("rows"))


@pytest.mark.parametrize("bath", [0, 2])
def test_rows_of_the_steps_before(exe, bath):
    r = subprocess.run([exe, str(bath)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    assert " 0 failures" in r.stdout
