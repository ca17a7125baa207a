"""The plan of a collection under a device-memory budget with the first tier's real limit (sets of up to 160 nodes), on the
CPU build of api.cpp: budgets a little above what the second query of 800 nodes needs with slices planned for sets of 128
nodes run that query; planned for 160, they would refuse it."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = "/opt/rocm/llvm/bin/clang++"


@pytest.mark.skipif(not os.path.exists(CLANG), reason="clang++ of the ROCm toolchain not found")
def test_budgets_near_the_smallest_that_runs(tmp_path):
    stub = open(os.path.join(ROOT, "tests/host_stub/launch_stub.cpp")).read()
    assert "? 128u : 512u" in stub
    (tmp_path / "launch_stub.cpp").write_text(stub.replace("? 128u : 512u", "? tim::kPoolSetCap : 512u"))
    exe = str(tmp_path / "budget_driver")
    subprocess.run([CLANG, "-std=c++17", "-O2", "-I", "tests/host_stub", "-I", "include", "-I",
                    "paper_1404_0900_amd/csrc", "paper_1404_0900_amd/csrc/api.cpp", "tests/host_stub/hip_stub.cpp",
                    str(tmp_path / "launch_stub.cpp"), "tests/host_stub/budget_driver.cpp", "-o", exe, "-lpthread"],
                   cwd=ROOT, check=True, capture_output=True, text=True)
    out = subprocess.run([exe, "607000", "630000", "1.01"], capture_output=True, text=True, timeout=300).stdout
    lines = [x for x in out.splitlines() if x.startswith("budget ")]
    assert len(lines) == 4 and all(": 1 of 4 ok, 0 differ" in x for x in lines), out
