"""The encode kernel of calls whose files have room for the longest stream (one kernel a call: a
workgroup a channel of a strip, its rows shared among the waves, its place in the file added up from what
the units ahead publish), compiled for the host and run on host threads under the sanitizers, byte for byte
the oracle's files.  Buffers are exactly the promised size: images end with their last pixel, files with
the bound that makes the calls take this kernel."""
import os
import struct

import numpy as np
import pytest

import oracle
from paper_2208_08711_amd import encode_bound, synth
from test_encoder_cpu_build import ASAN, build, exes, noise      # noqa: F401 (a fixture)
from test_kernel_cpu_build import ROOT, execute, run


def write_case(path, images, patches, calls=1, pads=(0,), room=lambda k, bound: bound):
    with open(path, "wb") as f:
        f.write(struct.pack("<3I", 0x4345334C, len(images), calls))
        for k, im in enumerate(images):
            patch = patches[k % len(patches)]
            want = oracle.encode(im, patch)
            h, w = im.shape[:2]
            f.write(struct.pack("<5IQ", w, h, patch, pads[k % len(pads)], k % 7, room(k, encode_bound(w, h, patch))))
            f.write(im.tobytes())
            f.write(struct.pack("<Q", len(want)))
            f.write(want)


def case_run(exes, kind, name, *args, **kw):                    # noqa: F811
    case = os.path.join(exes["tmp"], "chained_" + name + ".bin")
    write_case(case, *args, **kw)
    run(exes[kind], case)


@pytest.mark.parametrize("patch", [32, 64, 128])
def test_edges_of_lanes_waves_and_patches(exes, patch):         # noqa: F811
    """Last patches of 1 to 9 columns, images narrower than a lane's 12 bytes, heights around the rows of
    a wave (8 or 16) and of a reduction (4), patch rows of one row."""
    rows = 16 if patch == 128 else 8
    heights = [1, 2, 3, 4, 5, rows - 1, rows, rows + 1, 2 * rows + 3]
    images = [noise(900 + k, w, heights[k % 9]) for k, w in enumerate(list(range(1, 10)) + [patch + w for w in range(1, 10)])]
    images += [noise(930, patch + 3, patch + 1), noise(931, 256 + 5, 7)]
    case_run(exes, "asan", f"edges_{patch}", images, [patch], pads=(0, 5), calls=1)


@pytest.mark.parametrize("patch", [32, 64, 128])
def test_longest_and_shortest_streams(exes, patch):             # noqa: F811
    """Incompressible bytes fill the unit's bytes in LDS to the last; constant rows have no deltas; first
    rows of 0 to 8 bits, whose fields begin up to 4 bits ahead of the patch's bytes, beside other patches."""
    images = [noise(940, 256, patch), np.full((patch, 70, 3), 7, np.uint8)]
    for width in range(9):
        im = noise(950 + width, 2 * patch + 3, 5)
        im[0] = noise(970 + width, 2 * patch + 3, 1, 90, 90 + (1 << width))[0] if width < 8 else im[0]
        images.append(im)
    case_run(exes, "asan", f"streams_{patch}", images, [patch])


def test_calls_on_one_workspace_that_grows_and_counts_on(exes):  # noqa: F811
    """Later calls find the words of earlier ones in the workspace; mixed patch sizes are several launches;
    more than 32 images take the larger argument block, and have their words made ready."""
    images = [synth.cosine_field(980 + k, 60 + 9 * k, 40 + k) for k in range(5)]
    case_run(exes, "asan", "mixed", images, [32, 64, 128], calls=2)
    case_run(exes, "asan", "block", [noise(990 + k, 1 + k % 9, 1 + k % 6) for k in range(33)], [64])


def test_more_than_256_images_go_through_the_descriptor_table(exes):    # noqa: F811
    case_run(exes, "asan", "table", [noise(4000 + k, 1 + k % 3, 1 + k % 2) for k in range(257)], [32])


def sequence_run(exes, name, sequence, *args, **kw):            # noqa: F811
    case = os.path.join(exes["tmp"], "chained_" + name + ".bin")
    write_case(case, *args, **kw)
    r = execute(exes["asan"], case, sequence)
    assert r.returncode == 0, (sequence, r.stderr[-1500:])


@pytest.mark.parametrize("sequence", ["cere", "ecrer", "ecpepre"])
def test_captured_calls_and_ordinary_ones_of_one_context(exes, sequence):    # noqa: F811
    """c a call that is only recorded (the first of its context too: what is allocated then has not been
    cleared by anything that ran), r its replay, p a replay of which only the first workgroup has run yet,
    e an ordinary call: every file that is looked at is the oracle's."""
    images = [synth.cosine_field(1040, 70, 40), noise(1041, 300, 9)]
    sequence_run(exes, "capture_" + sequence, sequence, images, [32])


SOURCE = open(os.path.join(ROOT, "paper_2208_08711_amd", "csrc", "l3_encode.hip")).read()


@pytest.fixture(scope="module")
def few_looks(exes):                                            # noqa: F811
    """The same with waits that end after 8 looks (a look is slow on host threads), for images of any number of units."""
    old, most = "constexpr uint32_t kMaxLooks = 1u << 20;", "kMostUnitsOfOne[2] = {480, 640};"
    assert SOURCE.count(old) == 1 and SOURCE.count(most) == 1
    path = os.path.join(exes["tmp"], "l3_encode_few_looks.hip")
    with open(path, "w") as f:
        f.write(SOURCE.replace(old, "constexpr uint32_t kMaxLooks = 8;").replace(most, "kMostUnitsOfOne[2] = {3072, 3072};"))
    return dict(exes, asan=build(exes["tmp"], "encode_few_looks", ASAN, kernel_source=path))


def test_a_disturbed_word_is_right_again_a_launch_later(few_looks):
    """d takes tickets as launches that overlapped would; x is the call that finds the word so, and only that one
    is wrong.  Two patch sizes are two launches a call."""
    images = [synth.cosine_field(1050, 70, 40), noise(1051, 300, 9), noise(1052, 3, 3)]
    for sequence, patches in (("edxee", [32]), ("edxedxe", [32, 64, 32])):
        sequence_run(few_looks, "disturbed_" + sequence, sequence, images, patches)


def test_a_unit_that_is_not_written_shows_in_the_status_word(exes):    # noqa: F811
    """A copy of the source with few looks that takes an image's units from the last to the first: all but unit 0
    wait in vain, and unit 0, which clears the status word, is the last to run."""
    path = os.path.join(exes["tmp"], "l3_encode_reversed.hip")
    call = "encode_unit<N>(d, unit, units, number, &words[image], cells + (size_t)image * units_per_image + unit,"
    assert SOURCE.count(call) == 1
    with open(path, "w") as f:
        f.write(SOURCE.replace("constexpr uint32_t kMaxLooks = 1u << 20;", "constexpr uint32_t kMaxLooks = 8;")
                .replace(call, call.replace(" unit,", " units - 1 - unit,")))
    exe = build(exes["tmp"], "encode_reversed", ASAN, kernel_source=path)
    case = os.path.join(exes["tmp"], "chained_reversed.bin")
    write_case(case, [noise(1060, 300, 9)], [32])
    r = execute(exe, case)
    assert r.returncode == 1, r.stderr[-1500:]
    assert r.stderr.splitlines()[:2] == ["MISMATCH: length, image 0: 0", "MISMATCH: status, image 0: 4"], r.stderr[-1500:]


def test_the_numbers_of_launches_begin_again(exes):             # noqa: F811
    images = [synth.cosine_field(1050, 70, 40), noise(1051, 300, 9), noise(1052, 3, 3)]
    sequence_run(exes, "last_number", "eleeee", images, [32, 64, 32])


def test_one_file_without_that_room_takes_the_whole_call_to_the_other_kernels(exes):  # noqa: F811
    images = [synth.cosine_field(1000 + k, 70, 12) for k in range(3)]
    case_run(exes, "asan", "room", images, [32], room=lambda k, bound: bound - (k == 1))


def test_more_units_than_one_look_takes_in(few_looks):
    """522 units of one patch column: the last ones look 512 units back and find a total there or further.  (In a
    copy of the source that takes images of that many units whatever their patches.)"""
    case_run(few_looks, "asan", "long", [noise(1010, 1, 32 * 173 + 5)], [32])


@pytest.mark.parametrize("patch", [32, 64, 128])
def test_hand_overs_under_thread_sanitizer(exes, patch):        # noqa: F811
    case_run(exes, "tsan", f"tsan_{patch}", [noise(1020, patch + 5, 38), synth.cosine_field(1021, 70, 33)], [patch])


def test_planted_mistakes_are_seen(exes):                       # noqa: F811
    src = open(os.path.join(ROOT, "paper_2208_08711_amd", "csrc", "l3_encode.hip")).read()
    case = os.path.join(exes["tmp"], "chained_planted.bin")
    write_case(case, [noise(1030, 69, 37), noise(1031, 64, 64)], [64])
    for name, kind, old, new, report in [
            ("toolong", "asan", "    const uint32_t whole = unit_bytes / 16, tail", "    const uint32_t whole = unit_bytes / 16 + 300, tail",
             "buffer-overflow"),
            ("nobarrier", "tsan", "    if (xl == 0) wave_bits[wave][g] = bits;\n    __syncthreads();",
             "    if (xl == 0) wave_bits[wave][g] = bits;", "data race")]:
        assert src.count(old) == 1, name
        path = os.path.join(exes["tmp"], f"l3_encode_chained_{name}.hip")
        with open(path, "w") as f:
            f.write(src.replace(old, new))
        exe = build(exes["tmp"], f"encode_chained_{name}", ASAN if kind == "asan" else ["-fsanitize=thread"], kernel_source=path)
        r = execute(exe, case)
        assert r.returncode != 0 and report in r.stderr, (name, r.returncode, r.stderr[-1500:])
