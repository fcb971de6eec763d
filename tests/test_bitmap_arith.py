"""The bitmap's arithmetic on the CPU (tests/host/bitmap_check.hip), and the leaf
kernels' quotients next to whole numbers on the GPU
(tests/device/leaf_quot_check.hip)."""
import ctypes as C
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(HERE, "device", "libleafquot.so")


def test_bitmap_arithmetic(tmp_path):
    if shutil.which("hipcc") is None:
        pytest.skip("hipcc is absent")
    exe = tmp_path / "bitmap_check"
    subprocess.run(["hipcc", "-O2", "-std=c++17",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-w",
                    "-I", os.path.join(ROOT, "paper_1503_01839_amd", "csrc"),
                    os.path.join(HERE, "host", "bitmap_check.hip"), "-o", str(exe)],
                   check=True, capture_output=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "OK" in r.stdout, r.stdout + r.stderr


@pytest.mark.gpu
@pytest.mark.parametrize("seed", [1503, 1839])
def test_leaf_quotients_next_to_whole_numbers(pc, seed):
    if not os.path.exists(LIB):
        pytest.fail(f"{LIB} is missing: run __graft_entry__.build()")
    pc.lib()  # the HIP runtime the library uses is loaded first
    L = C.CDLL(LIB)
    L.pc_leaf_quot_check.argtypes = [C.c_uint64, C.c_uint64, C.c_void_p]
    L.pc_leaf_quot_check.restype = C.c_int
    out = (C.c_uint64 * 6)()
    print("case: leaf quotients, 10^8 pairs, seed", seed, flush=True)
    assert L.pc_leaf_quot_check(10**8, seed, out) == 0
    assert list(out[:4]) == [0, 0, 0, 0]
    # a random fraction is below 8 units of 2^-20, or raised to there, once in
    # 2^20 / 8; short divisors have whole quotients more often
    assert out[5] > 10**6 and out[4] < out[5] / 500
