"""Host code of the library (planner, programs, stream order, copies, launch
sizes) on a fake HIP runtime: no GPU needed, and what would fault or race on
one is an assertion here.  The checks are in host_runtime.py."""
import os
import shutil
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no host compiler")
    so = str(tmp_path_factory.mktemp("fake") / "libfakehip.so")
    subprocess.check_call([cxx, "-O1", "-std=c++17", "-shared", "-fPIC", os.path.join(HERE, "fake_hip.cpp"), "-o", so])
    return so


@pytest.mark.parametrize("check", ["growth", "batch_order", "batch_update", "marginal_launches", "tile_shapes", "capture"])
def test_host(fake, check):
    r = subprocess.run([sys.executable, os.path.join(HERE, "host_runtime.py"), fake, check], capture_output=True,
                       text=True, timeout=300)
    assert r.returncode == 0 and "ok " + check in r.stdout, r.stdout[-2000:] + r.stderr[-4000:]
