"""Builds a host-side test program (no GPU needed) that includes host_runtime.h,
against the built library."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2501_10946_amd")


def program(name, folder):
    hipcc = "/opt/rocm/bin/hipcc" if os.path.exists("/opt/rocm/bin/hipcc") else shutil.which("hipcc")
    if not hipcc:
        pytest.skip("hipcc not available")
    if not os.path.exists(os.path.join(PKG, "librbsog.so")):
        pytest.skip("librbsog.so is not built")
    exe = os.path.join(str(folder), name)
    subprocess.run([hipcc, "-O1", "-std=c++17", "--offload-arch=gfx950", "-Wno-unused-result",
                    f"-I{os.path.join(ROOT, 'include')}", f"-I{os.path.join(PKG, 'csrc')}",
                    os.path.join(ROOT, "tests", name + ".cpp"), "-o", exe, "-Wl,-E", f"-L{PKG}", "-lrbsog",
                    f"-Wl,-rpath,{PKG}"], check=True, capture_output=True)
    return exe
