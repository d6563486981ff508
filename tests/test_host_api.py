"""The host side of the C-ABI without a device: a small program
(tests/host/api_driver.cpp) linked against libfpts.so."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2501_12349_amd")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    from paper_2501_12349_amd import build, fpts
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not found")
    if not os.path.exists(fpts.LIB_PATH):
        build.build()
    d = tmp_path_factory.mktemp("host")
    obj, exe = str(d / "api_driver.o"), str(d / "api_driver")
    for cmd in ([hipcc, "-O1", "-std=c++17", "-x", "hip", "--offload-arch=gfx950",
                 "--offload-host-only", "-I", os.path.join(ROOT, "include"),
                 "-I", os.path.join(PKG, "csrc"), "-c",
                 os.path.join(ROOT, "tests", "host", "api_driver.cpp"), "-o", obj],
                [hipcc, "-rdynamic", obj, fpts.LIB_PATH, "-Wl,-rpath," + PKG, "-o", exe]):
        r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
        assert r.returncode == 0, "%s\n%s" % (" ".join(cmd), r.stderr[-4000:])
    return exe


def _run(driver, what):
    r = subprocess.run([driver, what], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, (r.stdout + r.stderr)[-6000:]


def test_workspace_sizes_never_decrease(driver):
    _run(driver, "sizes")


def test_workspaces_fit_the_budgets_they_fitted(driver):
    _run(driver, "budgets")


def test_device_setup_launches_of_large_meshes(driver):
    _run(driver, "setups")


def test_grids_are_multiples_of_the_xcd_count(driver):
    _run(driver, "grids")
