"""The fused call's write-out takes four columns a lane, counted from where the window's rows are aligned,
and up to three at each edge of a strip one by one: windows of every width modulo four at every column
modulo four, mirrored and not, narrower than four columns, and cut by the strips (256 columns) and the
patches at every place.  On the host threads under the sanitizers, and on the GPU.  Every bit against the
oracle."""
import os
import sys

import numpy as np
import pytest

import oracle
from paper_2208_08711_amd import synth

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
import test_kernel_cpu_build as host_build        # noqa: E402
from test_kernel_cpu_build import exes            # noqa: E402,F401


def windows(image_width, image_height, width, height):
    last = image_width - width
    columns = sorted({0, 1, 2, 3, last, max(0, last - 1), last // 2, min(last, 31), min(last, 130), min(last, 255)} & set(range(last + 1)))
    return [(x, (3 * k) % (image_height - height + 1), k & 1) for k, x in enumerate(columns)] + [(last, 0, 1), (0, 0, 1)]


@pytest.mark.parametrize("patch", [32, 64, 128])
def test_windows_on_host_threads(exes, patch):
    picture = synth.uniform_bytes(11, 300, 9)
    for width in (1, 3, 41, 254):
        crops = windows(300, 9, width, 6)[::3]
        case = os.path.join(exes["tmp"], f"columns_{patch}_{width}.bin")
        host_build.write_case(case, 2, [picture] * len(crops), patch, crops=crops, crop=(width, 6), dtype=width & 1)
        host_build.run(exes["asan"], case)


@pytest.mark.gpu
@pytest.mark.parametrize("patch", [32, 64, 128])
@pytest.mark.parametrize("width", [1, 2, 3, 4, 5, 7, 37, 126, 224, 254, 255, 257, 301])
def test_windows_on_the_gpu(patch, width):
    import torch
    import paper_2208_08711_amd as l3
    ctx = l3.Context(0)
    picture = synth.uniform_bytes(12, 543, 150)
    file = oracle.encode(picture, patch)
    device = torch.from_numpy(np.frombuffer(file, dtype=np.uint8).copy()).cuda()
    height, info = 133, l3.peek_header(file)
    for copies in (1, 60):              # few workgroups and many
        crops = windows(543, 150, width, height) * copies
        out = torch.full((len(crops), 3, height, width), -1, dtype=torch.int16, device="cuda")
        for first in range(0, len(crops), 250):
            part = crops[first:first + 250]
            l3.decode_crop_normalize_batch(ctx, [device] * len(part), [info] * len(part), part, width, height,
                                           synth.IMAGENET_MEAN, synth.IMAGENET_STD, out[first:first + len(part)])
        torch.cuda.synchronize()
        got = out.cpu().numpy().view(np.uint16)
        each = len(crops) // copies
        for k in range(each):
            x, y, flip = crops[k]
            want = oracle.crop_normalize(picture, x, y, flip, width, height, synth.IMAGENET_MEAN, synth.IMAGENET_STD, 0)
            assert np.array_equal(got[k], want), (x, y, flip)
        for k in range(each, len(crops)):
            assert np.array_equal(got[k], got[k - each]), crops[k]
    ctx.close()
