"""What the library enqueues, checked on the CPU: host_launches.cpp, linked with
the built library, stands in for the HIP runtime and records the launches."""
import os
import subprocess

import pytest

from paper_2609_38978_amd import park as P

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def _run(*cmd):
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, f"{' '.join(cmd)}\n{r.stdout}\n{r.stderr}"
    return r.stdout


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_launches_of_host_code(tmp_path):
    P.lib()  # built
    pkg = os.path.dirname(os.path.abspath(P.__file__))
    obj, exe = str(tmp_path / "host_launches.o"), str(tmp_path / "host_launches")
    _run(HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17", "-w", "-I",
         os.path.join(ROOT, "include"), "-c", os.path.join(ROOT, "tests", "host_launches.cpp"),
         "-o", obj)
    _run(HIPCC, obj, "-o", exe, os.path.join(pkg, "libpark.so"), "-Wl,-rpath," + pkg)
    assert "host launch checks passed" in _run(exe)
