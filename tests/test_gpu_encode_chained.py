"""The encode calls that are one kernel (few strips, files with room for the longest stream): byte for byte
the oracle's files around every edge of its split, from one workspace in any order of calls, replayed from a
graph, on two streams, and alike on both sides of the rule that picks it."""
import numpy as np
import pytest

import oracle
from paper_2208_08711_amd import synth
from test_gpu_encode import check, ctx, l3      # noqa: F401 (fixtures)

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def noise(seed, w, h, low=0, high=256):
    return np.random.default_rng(seed).integers(low, high, size=(h, w, 3)).astype(np.uint8)


def room_for(l3, images, patch):                # noqa: F811
    return [torch.full((l3.encode_bound(im.shape[1], im.shape[0], patch) + 8,), 0xAB, dtype=torch.uint8, device="cuda")
            for im in images]


def same(files, lens, status, images, patch):
    assert int(status.abs().sum()) == 0
    for k, im in enumerate(images):
        want, got = oracle.encode(im, patch), files[k].cpu().numpy()
        assert int(lens[k]) == len(want) and got[:len(want)].tobytes() == want, (k, im.shape)
        assert (got[len(want):] == 0xAB).all(), (k, im.shape)


@pytest.mark.parametrize("patch", [32, 64, 128])
def test_rows_around_the_waves_shares(l3, ctx, patch):          # noqa: F811
    """Heights around a wave's 8 or 16 rows, a reduction's 4 and the patch's end, widths around the
    unit's end; smooth, incompressible and constant."""
    heights = [1, 3, 4, 5, 7, 8, 9, 15, 16, 17, patch - 1, patch, patch + 1, patch + 17]
    widths = [1, 3, 4, 255, 256, 257, 256 + patch, 511, 2 * patch - 2, patch + 1, 64, 33, 130, 300]
    images = [noise(2500 + k, w, h) if k % 2 else synth.cosine_field(2500 + k, w, h) for k, (w, h) in enumerate(zip(widths, heights))]
    images.append(np.full((patch + 5, 260, 3), 9, np.uint8))
    check(l3, ctx, images, patch=patch, pad_cols=1)


def test_many_units_of_one_image(l3, ctx):                      # noqa: F811
    """Up to the most units a call of one image takes, where a unit looks back more than once: 1024 counted
    ones and, with more than 4096 patches, 3072."""
    check(l3, ctx, [noise(2600, 3, 32 * 511)], patch=32)
    check(l3, ctx, [noise(2601, 70, 64 * 341)], patch=64)
    check(l3, ctx, [noise(2602, 32 * 48, 32 * 100, 0, 9)], patch=32)


@pytest.mark.parametrize("patch,strips,most", [(32, 4, 40), (64, 7, 30), (64, 3, 71)])
def test_both_sides_of_the_rule_for_one_image(l3, ctx, patch, strips, most):    # noqa: F811
    """Images of at most 480 units at N = 32 and 640 at N = 64 take the one kernel, longer ones the strip kernel, and
    those of more than 4096 patches the one kernel again."""
    for rows in (most, most + 1):
        check(l3, ctx, [noise(2650 + rows, 255 * strips, patch * rows - 3, 0, 30)], patch=patch)
    check(l3, ctx, [noise(2660, 64 * 40, 64 * 35, 0, 9)], patch=64)


@pytest.mark.parametrize("patch,shape,most", [(32, (500, 375), 21), (64, (640, 500), 14), (128, (700, 500), 28)])
def test_both_sides_of_the_rule(l3, ctx, patch, shape, most):   # noqa: F811
    """`most` images of 72 (N = 32), 72 and 36 units are the last that the rule's 1536 and 1024 units hold."""
    distinct = [noise(2700 + k, *shape, 0, 40 + k) for k in range(3)]
    for n in (most, most + 1):
        images = [distinct[k % 3] for k in range(n)]
        dev = [torch.from_numpy(im).cuda() for im in images]
        files = room_for(l3, images, patch)
        lens, status = torch.zeros(n, dtype=torch.int64, device="cuda"), torch.full((n,), 7, dtype=torch.int32, device="cuda")
        l3.encode_batch(ctx, dev, files, lens, patch=patch, status=status)
        torch.cuda.synchronize()
        same(files, lens, status, images, patch)


def test_one_workspace_grows_and_serves_calls_of_every_kind(l3):    # noqa: F811
    own = l3.Context(0)
    for k in range(3):
        check(l3, own, [noise(2800 + k, 100, 90)], patch=32)
        check(l3, own, [synth.cosine_field(2810 + k, 700, 600 + k)], patch=64)
        check(l3, own, [noise(2820 + i, 40 + i, 30 + k) for i in range(40)], patch=32)
        check(l3, own, [noise(2830 + i, 300, 200) for i in range(3)], patch=[128, 32, 64])
        check(l3, own, [noise(2840 + k, 200, 64 * 200)], patch=64)
    own.close()


def test_calls_in_a_row_and_on_two_streams_without_waiting(l3, ctx):    # noqa: F811
    """Forty calls of different inputs on one context, every other one on a second stream, all waited
    for once at the end."""
    images = [synth.cosine_field(2900 + k, 400 + 3 * k, 300 + k) for k in range(4)]
    dev = [torch.from_numpy(im).cuda() for im in images]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    kept = []
    for call in range(40):
        order = [(call + k) % 4 for k in range(1 + call % 4)]
        batch = [images[i] for i in order]
        with torch.cuda.stream(streams[call % 2]):
            files = room_for(l3, batch, 32)
            lens, status = torch.zeros(len(batch), dtype=torch.int64, device="cuda"), torch.zeros(len(batch), dtype=torch.int32, device="cuda")
            l3.encode_batch(ctx, [dev[i] for i in order], files, lens, patch=32, status=status)
        kept.append((files, lens, status, batch))
    torch.cuda.synchronize()
    for files, lens, status, batch in kept:
        same(files, lens, status, batch, 32)


def test_replayed_from_a_captured_graph(l3):                    # noqa: F811
    """Every replay reads new pixels, with eager calls of the same context between the replays."""
    own = l3.Context(0)
    images = [synth.cosine_field(3000 + k, 333, 210) for k in range(3)]
    dev = [torch.from_numpy(im).cuda() for im in images]
    files = room_for(l3, images, 64)
    lens, status = torch.zeros(3, dtype=torch.int64, device="cuda"), torch.zeros(3, dtype=torch.int32, device="cuda")
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        l3.encode_batch(own, dev, files, lens, patch=64, status=status)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        l3.encode_batch(own, dev, files, lens, patch=64, status=status)
    for rep in range(4):
        print(f"graph replay {rep}", flush=True)
        now = [np.roll(im, 17 * rep + k, axis=1) for k, im in enumerate(images)]
        for d, im in zip(dev, now):
            d.copy_(torch.from_numpy(np.ascontiguousarray(im)))
        for f in files:
            f.fill_(0xAB)
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            graph.replay()
        torch.cuda.synchronize()
        same(files, lens, status, now, 64)
        other = room_for(l3, images[:1], 32)
        with torch.cuda.stream(side):
            l3.encode_batch(own, dev[:1], other, lens[:1], patch=32, status=status[:1])
        torch.cuda.synchronize()
        same(other, lens, status, now[:1], 32)
    own.close()


@pytest.mark.parametrize("mode", ["global", "relaxed"])
def test_captured_before_the_workspace_has_served_such_a_call(l3, mode):    # noqa: F811
    """A small call is captured when its context has served one large call only (the default mode allows no
    allocation), or none (relaxed mode).  Ordinary small calls ahead of the first replay and between the replays."""
    own = l3.Context(0)
    image = synth.cosine_field(3100, 333, 210)
    dev, files = torch.from_numpy(image).cuda(), room_for(l3, [image], 64)
    lens, status = torch.zeros(1, dtype=torch.int64, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
    side = torch.cuda.Stream()
    if mode == "global":
        many = [noise(3110 + k % 3, 500, 375, 0, 60) for k in range(30)]
        large, n = room_for(l3, many, 32), len(many)
        all_lens, all_status = torch.zeros(n, dtype=torch.int64, device="cuda"), torch.zeros(n, dtype=torch.int32, device="cuda")
        large_dev = [torch.from_numpy(im).cuda() for im in many]
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            l3.encode_batch(own, large_dev, large, all_lens, patch=32, status=all_status)
        torch.cuda.synchronize()
        same(large, all_lens, all_status, many, 32)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side, capture_error_mode=mode):
        l3.encode_batch(own, [dev], files, lens, patch=64, status=status)
    for rep in range(4):
        print(f"{mode} {rep}", flush=True)
        other = room_for(l3, [image], 32)
        with torch.cuda.stream(side):
            l3.encode_batch(own, [dev], other, lens, patch=32, status=status)
        torch.cuda.synchronize()
        same(other, lens, status, [image], 32)
        files[0].fill_(0xAB)
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            graph.replay()
        torch.cuda.synchronize()
        same(files, lens, status, [image], 64)
    own.close()


@pytest.mark.parametrize("patch,height", [(32, 30), (64, 40), (128, 40)])
def test_more_images_than_the_arguments_hold(l3, ctx, patch, height):    # noqa: F811
    """300 images, whose descriptors come from the table in device memory: with room for the longest stream one
    kernel, with room for exactly their files the strip and copy kernels."""
    distinct = [noise(3200 + k, 60 - k, height - k % 3, 0, 30 + 9 * k) for k in range(7)]
    images = [distinct[k % 7] for k in range(300)]
    dev = [torch.from_numpy(distinct[k]).cuda() for k in range(7)]
    exact = [torch.full((len(oracle.encode(distinct[k % 7], patch)),), 0xAB, dtype=torch.uint8, device="cuda") for k in range(300)]
    for files in (room_for(l3, images, patch), exact):
        lens, status = torch.zeros(300, dtype=torch.int64, device="cuda"), torch.full((300,), 7, dtype=torch.int32, device="cuda")
        l3.encode_batch(ctx, [dev[k % 7] for k in range(300)], files, lens, patch=patch, status=status)
        torch.cuda.synchronize()
        same(files, lens, status, images, patch)
