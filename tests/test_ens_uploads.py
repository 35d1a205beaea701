"""Uploads of the served ensemble (host only, no GPU): around the 4 MiB of pinned
memory that admissions send from.  64 bytes a particle go up beside the tables:
1 000 and 60 000 fit, of 65 400 (4 185 600 bytes) the tables do not all fit, of
87 000 the charges do not, of 200 000 nothing of the state does."""
import subprocess

import pytest

from host_runtime import program


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    return program("ens_uploads_check", tmp_path_factory.mktemp("uploads"))


@pytest.mark.parametrize("N", [1000, 60000, 65400, 87000, 200000])
def test_sources_outlive_their_copies(exe, N):
    r = subprocess.run([exe, str(N)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "0 failures" in r.stdout
