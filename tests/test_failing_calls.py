"""What a call that failed part way leaves for the next one: the host planner on
a stand-in device whose allocations fail on demand (tests/host/failing_calls.hip)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    if shutil.which("hipcc") is None:
        pytest.skip("hipcc is absent")
    out = tmp_path_factory.mktemp("host") / "failing_calls"
    subprocess.run(["hipcc", "-O1", "-std=c++17", "--offload-arch=gfx950",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-w",
                    "-I", os.path.join(ROOT, "paper_1503_01839_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "failing_calls.hip"), "-o", str(out)],
                   check=True, capture_output=True)
    return str(out)


@pytest.mark.parametrize("case", ["tables", "batch", "seeds"])
def test_next_call_after_a_failure(exe, case):
    r = subprocess.run([exe, case], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "OK" in r.stdout, r.stdout + r.stderr
