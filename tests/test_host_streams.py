"""What the C ABI's calls allocate and which wait for each other on the host, with the
HIP runtime's calls replaced (tests/host_streams.cpp): no GPU is used."""
import os
import subprocess

import pytest

from tests.conftest import ROOT

psflib = pytest.importorskip("paper_2106_09122_amd.psflib")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host") / "host_streams")
    pkg = os.path.dirname(psflib.LIB_PATH)
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-D__HIP_PLATFORM_AMD__=1", "-I", os.path.join(ROOT, "include"),
                        "-isystem", "/opt/rocm/include", os.path.join(ROOT, "tests", "host_streams.cpp"),
                        "-L", pkg, "-l:" + os.path.basename(psflib.LIB_PATH), "-L/opt/rocm/lib", "-lamdhip64",
                        "-rdynamic", "-pthread", "-Wl,-rpath," + pkg, "-Wl,-rpath,/opt/rocm/lib", "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return exe


@pytest.mark.parametrize("what", ["memory", "streams"])
def test_host_streams(driver, what):
    r = subprocess.run([driver, what], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "host_streams ok" in r.stdout, (r.stdout[-2000:], r.stderr[-2000:])
