"""Storing H with host memory short: the plan of tiles needs some, H itself does not.
A C++ client refuses large host allocations while H is stored; no exception may leave
the C entry point, and H serves without a plan."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2509_26309_amd")
SRC = os.path.join(ROOT, "tests", "c_client", "tbpm_host_memory.cpp")


@pytest.fixture(scope="module")
def client(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("g++ not found")
    if not os.path.exists(os.path.join(PKG, "libtbpm.so")):
        pytest.fail("libtbpm.so is not built")
    exe = str(tmp_path_factory.mktemp("host_memory") / "tbpm_host_memory")
    cmd = ["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-I", os.path.join(ROOT, "include"), SRC, "-o", exe,
           "-L", PKG, "-ltbpm", "-Wl,-rpath," + PKG]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr
    return exe


def test_client_builds(client):
    assert os.access(client, os.X_OK)


@pytest.mark.gpu
@pytest.mark.parametrize("fmt", [1, 2], ids=["ell", "uneven_csr"])
def test_no_plan_without_host_memory(client, fmt):
    r = subprocess.run([client, str(fmt)], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stdout + r.stderr
    assert r.stdout.count(": ok") == 9 and "FAILED" not in r.stdout, r.stdout
