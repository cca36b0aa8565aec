"""The encode kernels' own source (paper_2208_08711_amd/csrc/l3_encode.hip with its host planning)
compiled for the host and run on host threads, one per GPU thread (tests/native/kernel_cpu), under
AddressSanitizer + UBSan and under ThreadSanitizer: every file byte for byte the oracle's, images
and files in buffers of exactly their size (a lane reads 12 bytes of a row at a time, without a
condition), every hand-over through LDS, the size table and the slots ordered.  No GPU; the same
kernels run on the GPU in tests/test_gpu_encode.py."""
import os
import struct
import subprocess
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

import oracle
from paper_2208_08711_amd import synth
from test_kernel_cpu_build import CLANG, ROOT, execute, run

SOURCES = [os.path.join(ROOT, "tests", "native", "kernel_cpu", "encode_cpu_main.cpp"),
           os.path.join(ROOT, "paper_2208_08711_amd", "csrc", "l3_host.cpp")]
ASAN = ["-fsanitize=address,undefined", "-fno-sanitize-recover=undefined"]


def build(tmp, name, flags, kernel_source=None):
    exe = os.path.join(tmp, name)
    if kernel_source:
        flags = [*flags, f'-DL3_KERNEL_SOURCE="{kernel_source}"']
    subprocess.run([CLANG, "-std=c++17", "-O1", "-g", "-ffp-contract=off", "-pthread", *flags,
                    "-I", os.path.join(ROOT, "tests", "native", "kernel_cpu"),
                    "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2208_08711_amd", "csrc"),
                    "-x", "c++", *SOURCES, "-o", exe], check=True)
    return exe


@pytest.fixture(scope="module")
def exes(tmp_path_factory):
    if not os.path.exists(CLANG):
        pytest.skip("no clang++ with sanitizer runtimes")
    tmp = str(tmp_path_factory.mktemp("encode_cpu"))
    with ThreadPoolExecutor(2) as pool:
        asan = pool.submit(build, tmp, "encode_cpu_asan", ASAN)
        tsan = pool.submit(build, tmp, "encode_cpu_tsan", ["-fsanitize=thread"])
        return {"asan": asan.result(), "tsan": tsan.result(), "tmp": tmp}


def write_case(path, images, patches, calls=1, pads=(0,), short=()):
    """pads: bytes between the rows, in turn; short: images whose file buffer is a byte too small
    (odd ones of them: too small for the header as well)."""
    with open(path, "wb") as f:
        f.write(struct.pack("<3I", 0x4345334C, len(images), calls))
        for k, im in enumerate(images):
            patch = patches[k] if isinstance(patches, list) else patches
            want = oracle.encode(im, patch)
            assert np.array_equal(oracle.decode(want), im)
            h, w = im.shape[:2]
            cap = len(want)
            if k in short:
                cap = cap - 1 if k % 2 == 0 else 12
            f.write(struct.pack("<5IQ", w, h, patch, pads[k % len(pads)], k % 7, cap))
            f.write(im.tobytes())
            f.write(struct.pack("<Q", len(want)))
            f.write(want)


def case_run(exes, kind, name, *args, **kw):
    case = os.path.join(exes["tmp"], name + ".bin")
    write_case(case, *args, **kw)
    run(exes[kind], case)


def noise(seed, w, h, low=0, high=256):
    return np.random.default_rng(seed).integers(low, high, size=(h, w, 3)).astype(np.uint8)


@pytest.mark.parametrize("patch", [32, 64, 128])
def test_last_lanes_and_rows_of_every_width_and_height(exes, patch):
    """Last patches of 1 to 9 columns (a lane at the edge steps back so as not to read past the
    row), images narrower than one lane's 12 bytes, 1 to 5 rows (rows that do not exist repeat the
    last one), rows right behind one another and with a gap."""
    shapes = [(w, 1 + w % 5) for w in range(1, 10)] + [(patch + w, 1 + (w + 2) % 5) for w in range(1, 10)]
    shapes += [(256 + 3, 9)]
    images = [noise(100 + k, w, h) for k, (w, h) in enumerate(shapes)]
    case_run(exes, "asan", f"edges_{patch}", images, patch, pads=(0, 5))


@pytest.mark.parametrize("patch", [32, 64, 128])
def test_full_patches_of_incompressible_bytes(exes, patch):
    """The longest stream there is: the ring carries its largest backlog from period to period;
    a strip has lanes without a patch beside it, and a last patch row of one row."""
    images = [noise(200, patch, patch), noise(201, patch + 6, patch + 1)]
    case_run(exes, "asan", f"full_{patch}", images, patch)


@pytest.mark.parametrize("patch", [32, 64, 128])
def test_widths_of_the_first_rows(exes, patch):
    """The first record's deltas of 0 to 8 bits are put into the ring from up to 4 bits ahead of the
    stream (its last word and the word behind it), then rows of other widths."""
    images = []
    for width in range(9):
        im = noise(300 + width, patch + 3, 6)
        im[0] = noise(320 + width, patch + 3, 1, 90, 90 + (1 << width))[0] if width < 8 else im[0]
        images.append(im)
    case_run(exes, "asan", f"first_{patch}", images, patch)


def test_constant_and_smooth_content_several_calls_on_one_workspace(exes):
    images = [np.full((40, 70, 3), 255, np.uint8), np.zeros((33, 5, 3), np.uint8), synth.cosine_field(11, 75, 36)]
    for patch in (32, 64, 128):
        case_run(exes, "asan", f"calls_{patch}", images, patch, calls=2)


def test_all_patch_sizes_and_both_routes_in_one_call(exes):
    """With an image on the plain route the layout kernel works the offsets out for all."""
    images = [synth.cosine_field(20 + k, 67 + k, 20 + k) for k in range(5)]
    case_run(exes, "asan", "mixed", images[:4], [32, 64, 128, 32])
    case_run(exes, "asan", "routes", images[:4] + [noise(400, 15, 9)], [32, 64, 128, 33, 7])
    case_run(exes, "asan", "plain", [noise(401, 2, 3), noise(402, 131, 9), noise(403, 100, 101)], [1, 128 - 1, 100])


def test_more_than_32_images_take_the_larger_argument_block(exes):
    images = [noise(500 + k, 1 + k % 9, 1 + k % 6) for k in range(33)]
    case_run(exes, "asan", "block", images, 64, calls=2)
    case_run(exes, "asan", "table_plain", images, [(32, 9)[k % 2] for k in range(33)])


@pytest.mark.parametrize("patch", [32, 64, 128])
def test_more_than_256_images_go_through_the_descriptor_table(exes, patch):
    case_run(exes, "asan", f"table_{patch}", [noise(5000 + k, 1 + k % 3, 1 + k % 2) for k in range(257)], patch)


def test_files_without_room_receive_their_header_only(exes):
    images = [synth.cosine_field(600 + k, 70, 12) for k in range(6)]
    case_run(exes, "asan", "short", images, [32, 32, 64, 64, 128, 128], short=(0, 1, 2, 3, 4, 5))
    case_run(exes, "asan", "short_plain", images[:4], [32, 32, 50, 50], short=(0, 1, 2, 3))


@pytest.mark.parametrize("patch", [32, 64, 128, 100])
def test_hand_overs_under_thread_sanitizer(exes, patch):
    case_run(exes, "tsan", f"tsan_{patch}", [noise(700, 2 * patch + 5, 38), synth.cosine_field(701, 70, 33)], patch)


def test_planted_mistakes_are_seen(exes):
    """Copies of the kernel source with one mistake each: an edge lane that does not step back, a
    ring flushed without its fence, a slot copied one granule too far."""
    src = open(os.path.join(ROOT, "paper_2208_08711_amd", "csrc", "l3_encode.hip")).read()
    case = os.path.join(exes["tmp"], "planted.bin")
    write_case(case, [noise(800, 69, 37), noise(801, 64, 64)], 64)
    plants = [
        ("stepback", "asan", "const uint32_t back = wide && nvalid ? 3 * (4 - nvalid) : 0;",
         "const uint32_t back = 0;", "heap-buffer-overflow"),
        ("nofence", "tsan", "    auto flush = [&](uint32_t end) {\n        wave_lds_fence();",
         "    auto flush = [&](uint32_t end) {", "data race"),
        ("toofar", "asan", "        whole[j] = bytes / 16;", "        whole[j] = bytes / 16 + 1;", "heap-buffer-overflow"),
    ]

    def build_plant(plant):
        name, kind, old, new, report = plant
        assert src.count(old) == 1, name
        path = os.path.join(exes["tmp"], f"l3_encode_{name}.hip")
        with open(path, "w") as f:
            f.write(src.replace(old, new))
        return build(exes["tmp"], f"encode_cpu_{name}", ASAN if kind == "asan" else ["-fsanitize=thread"], kernel_source=path)

    with ThreadPoolExecutor(3) as pool:
        built = list(pool.map(build_plant, plants))
    for (name, kind, old, new, report), exe in zip(plants, built):
        r = execute(exe, case)
        assert r.returncode != 0 and report in r.stderr, (name, r.returncode, r.stderr[-1500:])
