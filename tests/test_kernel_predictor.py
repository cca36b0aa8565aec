"""The predictor of the decode and encode kernels works on packed 16-bit floats.  Its own source,
built for the host (tests/native/kernel_cpu), against the definition of arxiv 2208.08711
Section 4.2 for every value of the three neighbours, in inner, first and last columns.  No GPU;
what the instructions themselves do is checked by the exhaustive cases of
tests/test_gpu_parity.py and tests/test_gpu_encode.py."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = "/opt/rocm/llvm/bin/clang++"
HERE = os.path.join(ROOT, "tests", "native", "kernel_cpu")


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    if not os.path.exists(CLANG):
        pytest.skip("no clang++")
    out = str(tmp_path_factory.mktemp("predictor") / "predictor")
    subprocess.run([CLANG, "-std=c++17", "-O2", "-ffp-contract=off", "-pthread", "-I", HERE,
                    "-I", os.path.join(ROOT, "paper_2208_08711_amd", "csrc"), "-x", "c++",
                    os.path.join(HERE, "predictor_main.cpp"), "-o", out], check=True)
    return out


@pytest.mark.parametrize("first", [0, 64, 128, 192])
def test_prediction_is_the_nearest_neighbour_for_all_values(exe, first):
    r = subprocess.run([exe, str(first), str(first + 64)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout == "ok\n", (r.stdout, r.stderr[-2000:])
