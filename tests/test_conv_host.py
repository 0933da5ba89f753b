"""The convolution form of the M2L (csrc/k_conv.hip) on the host: its index
maps hit every array entry once, and its blocks, columns and transforms in plain
loops (tests/host/conv_check.cpp, on the header the kernels include) give the sum
over the 875 offsets of every cell."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2003_13218_amd", "csrc")


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    exe = str(tmp_path_factory.mktemp("conv") / "conv_check")
    src = [os.path.join(ROOT, "tests", "host", "conv_check.cpp"), os.path.join(CSRC, "conv_layout.cpp"),
           os.path.join(CSRC, "harmonics_host.cpp")]
    r = subprocess.run([hipcc, "-O2", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I", CSRC, *src, "-o", exe,
                        "-lpthread"], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]

    def run(*args):
        return subprocess.run([exe, *map(str, args)], capture_output=True, text=True, timeout=300)
    return run


@pytest.mark.parametrize("level", [1, 2, 3, 4, 5, 6])
@pytest.mark.parametrize("p", [0, 3, 4, 9])
def test_maps_hit_every_entry_once(check, level, p):
    r = check("maps", level, p)
    assert (r.returncode, r.stdout.strip()) == (0, "ok")


@pytest.mark.parametrize("level,p", [(1, 0), (1, 4), (2, 3), (2, 6), (3, 2)])
def test_convolution_is_the_sum_over_the_list(check, level, p):
    # two FP64 sums of at most 875 K terms of size <= 1/3 each, relative to the
    # largest result: 1e-16 times the square root of their number times 100
    r = check("sum", level, p)
    assert r.returncode == 0 and float(r.stdout) < 1e-16 * 100 * (875 * (p + 1) ** 2) ** 0.5, r.stdout
