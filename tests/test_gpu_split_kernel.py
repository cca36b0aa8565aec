"""Launches around the bound between the split kernels and the ones of three waves (two workgroups a
compute unit): on both sides of it, for every patch size and layout, with ragged edges, words of the status,
damaged streams and replays of a captured graph.  Every byte against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2208_08711_amd as l3
from paper_2208_08711_amd import synth

pytestmark = pytest.mark.gpu


def decode(ctx, files, layout, repeat=1, stream=None):
    infos = [l3.peek_header(f) for f in files]
    device = [torch.from_numpy(np.frombuffer(f, dtype=np.uint8).copy()).cuda() for f in files]
    shapes = [(3, i.height, i.width) if layout == l3.LAYOUT_CHW else (i.height, i.width, 3) for i in infos]
    outs = [torch.full(s, 0xA5, dtype=torch.uint8, device="cuda") for s in shapes * repeat]
    status = torch.full((len(outs),), 77, dtype=torch.int32, device="cuda")
    l3.decode_batch(ctx, device * repeat, infos * repeat, outs, layout=layout, status=status)
    torch.cuda.synchronize()
    return [o.cpu().numpy() for o in outs], status.cpu().numpy()


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("patch", [32, 64, 128])
def test_both_sides_of_the_bound(patch, layout):
    """Images of 3 patch rows and a rest each; 504 to 528 units of work (the bound is 512 on 256 CUs)."""
    ctx = l3.Context(0)
    height = 3 * patch + 5
    pictures = [synth.cosine_field(9, 256 + 3, height), synth.uniform_bytes(10, 256 + 130, height)]
    files = [oracle.encode(p, patch) for p in pictures]
    want = [oracle.decode(f) for f in files]
    for repeat in (1, 30, 32, 33, 40):
        outs, status = decode(ctx, files, layout, repeat)
        assert not status.any()
        for k, out in enumerate(outs):
            w = want[k % 2]
            assert np.array_equal(out, w.transpose(2, 0, 1) if layout else w), (repeat, k)
    ctx.close()


@pytest.mark.parametrize("patch", [32, 64, 128])
def test_every_number_of_rows(patch):
    """Patches of 1 to 14 rows and around the ends of periods of six: whole periods, rests, neither."""
    ctx = l3.Context(0)
    rows = [h for h in (*range(1, 15), 17, 18, 19, 29, 30, 31, 63, 64, 65, 125, 126, 127, 128) if h <= patch]
    pictures = [synth.uniform_bytes(40 + h, 2 * patch + 1 + h % 5, h) for h in rows]
    files = [oracle.encode(p, patch) for p in pictures]
    for layout in (0, 1):
        outs, status = decode(ctx, files, layout)
        assert not status.any()
        for out, p in zip(outs, pictures):
            assert np.array_equal(out, p.transpose(2, 0, 1) if layout else p), p.shape
    ctx.close()


def test_status_words_of_a_damaged_stream():
    """A width above 8 and a stream that ends early are flagged, the neighbours' words and pixels are not
    touched: an image of one unit of work (its word is stored) and one of many (flags are ORed in)."""
    ctx = l3.Context(0)
    for width in (200, 900):
        picture = synth.uniform_bytes(3, width, 130)
        good = oracle.encode(picture, 64)
        header = l3.peek_header(np.frombuffer(good, dtype=np.uint8)).header_bytes
        bad = bytearray(good)
        bad[header] = (bad[header] & 0xF0) | 15
        outs, status = decode(ctx, [good, bytes(bad), good], 0)
        assert status[0] == 0 and status[2] == 0 and status[1] & 1
        assert np.array_equal(outs[0], picture) and np.array_equal(outs[2], picture)
    ctx.close()


def test_replays_of_a_captured_graph():
    ctx = l3.Context(0)
    picture = synth.voronoi_scene(4, 700, 300)
    file = oracle.encode(picture, 64)
    info = l3.peek_header(file)
    device = torch.from_numpy(np.frombuffer(file, dtype=np.uint8).copy()).cuda()
    out = torch.zeros(picture.shape, dtype=torch.uint8, device="cuda")
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    l3.decode_batch(ctx, [device], [info], [out], status=status)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        l3.decode_batch(ctx, [device], [info], [out], status=status)
    for _ in range(4):
        out.fill_(7)
        status.fill_(9)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert int(status[0]) == 0 and np.array_equal(out.cpu().numpy(), picture)
        l3.decode_batch(ctx, [device], [info], [out], status=status)
    ctx.close()
