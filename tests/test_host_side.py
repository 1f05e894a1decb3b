"""The host side of a run (pdfs_api.cpp), compiled against stand-ins for the HIP
calls and the launches (tests/host/stub.h).  alloc: device memory runs out, and
every buffer that a launch is handed has to be held and long enough; memory:
counters that nobody asked for, lists that do not fit; routes: lazy or walked
rounds.  No GPU."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2603_16721_amd", "csrc")


@pytest.mark.parametrize("name", ["alloc", "memory", "routes"])
def test_host(tmp_path, name):
    exe = str(tmp_path / name)
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-w",
                    "-I/opt/rocm/include", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    os.path.join(ROOT, "tests", "host", name + ".cpp"),
                    os.path.join(CSRC, "pdfs_api.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.startswith("ok"), (r.returncode, r.stdout)
