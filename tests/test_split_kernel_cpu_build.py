"""The decode kernels for launches of few workgroups (l3_decode_split_kernel_args: records and deltas,
filter and write-out by different waves) as source on host threads, under AddressSanitizer + UBSan and
ThreadSanitizer, and as compiled, in the interpreter.  The host build takes them when its stand-in for the
runtime reports many compute units (L3CPU_CUS).  Every byte against the oracle.  No GPU."""
import os
import re
import struct
import subprocess
import sys

import pytest

from paper_2208_08711_amd import synth

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
import test_kernel_cpu_build as host_build        # noqa: E402
import test_kernel_machine_code as machine_code   # noqa: E402
from test_kernel_cpu_build import exes            # noqa: E402,F401
from test_kernel_machine_code import built        # noqa: E402,F401


@pytest.fixture(autouse=True)
def many_compute_units(monkeypatch):
    monkeypatch.setenv("L3CPU_CUS", "256")


# rows: one, a period of four less, exactly and more, several periods, whole patches, more than one patch row
SHAPES = [(1, 1), (3, 5), (65, 4), (5, 3), (33, 31), (130, 8), (257, 9), (63, 65), (129, 66)]


def images(seed):
    return [synth.cosine_field(seed + k, w, h) if k % 2 else synth.uniform_bytes(seed + k, w, h)
            for k, (w, h) in enumerate(SHAPES)]


@pytest.mark.parametrize("patch", [32, 64, 128])
@pytest.mark.parametrize("mode", [0, 1])
def test_pixel_modes_under_address_and_ub_sanitizers(exes, patch, mode):
    case = os.path.join(exes["tmp"], f"split_px_{patch}_{mode}.bin")
    host_build.write_case(case, mode, images(700 + patch) + [synth.uniform_bytes(5, 140, 133)], patch)
    host_build.run(exes["asan"], case)


@pytest.mark.parametrize("patch", [32, 64, 128])
def test_fused_path_under_address_and_ub_sanitizers(exes, patch):
    pictures = [synth.cosine_field(40 + k, 70 + 9 * k, 50 + 7 * k) for k in range(4)]
    crops = [(0, 0, 0), (7, 3, 1), (79 - 40, 57 - 33, 0), (31, 17, 1)]
    for mode, dtype in ((2, 0), (3, 1)):
        case = os.path.join(exes["tmp"], f"split_fused_{patch}_{mode}.bin")
        host_build.write_case(case, mode, pictures, patch, crops=crops, crop=(40, 33), dtype=dtype)
        host_build.run(exes["asan"], case)


def test_more_than_32_images(exes):
    case = os.path.join(exes["tmp"], "split_many.bin")
    host_build.write_case(case, 0, [synth.uniform_bytes(3000 + k, 1 + k % 7, 1 + k % 5) for k in range(40)], 32)
    host_build.run(exes["asan"], case)


@pytest.mark.parametrize("patch,mode", [(32, 0), (64, 0), (128, 0), (64, 1), (32, 2)])
def test_lds_protocol_under_thread_sanitizer(exes, patch, mode):
    """Values, parked rows and the table are handed between the waves at one barrier a period."""
    pictures = [synth.cosine_field(70, 140, 75), synth.uniform_bytes(71, 66, 40)]
    case = os.path.join(exes["tmp"], f"split_tsan_{patch}_{mode}.bin")
    if mode == 2:
        host_build.write_case(case, 2, pictures, patch, crops=[(10, 5, 1), (3, 2, 0)], crop=(50, 30))
    else:
        host_build.write_case(case, mode, pictures, patch)
    host_build.run(exes["tsan"], case)


@pytest.mark.parametrize("patch,mode", [(32, 0), (64, 0), (128, 0), (32, 1), (64, 1), (128, 1), (32, 2), (128, 2)])
def test_kernels_as_compiled(built, monkeypatch, patch, mode):
    def text(asm, n, kmode, kind):
        assert kind in (3, 4)
        name = "_ZN12_GLOBAL__N_127l3_decode_split_kernel_argsILi%dELi%dELi%dEEE" % (n, kmode, 32 if kind == 3 else 256)
        m = re.search(r"^" + re.escape(name) + r"\S*: +; @", asm, flags=re.M)
        assert m, name
        return asm[m.start():asm.index(".end_amdhsa_kernel", m.start())]
    monkeypatch.setattr(machine_code, "kernel_text", text)
    if mode == 2:
        pictures = [synth.cosine_field(50 + k, 70 + 9 * k, 50 + 7 * k) for k in range(2)]
        machine_code.record_and_interpret(built, f"split_{patch}_{mode}", mode, pictures, patch,
                                          crops=[(7, 3, 1), (20, 11, 0)], crop=(40, 33), dtype=0)
    else:
        machine_code.record_and_interpret(built, f"split_{patch}_{mode}", mode, machine_code.small_images(300 + patch), patch)
