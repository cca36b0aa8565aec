"""The work that a user of this library has it do, as cases that can be timed and compared.

Three directions: decode files to 8-bit RGB (interleaved or planar), decode a window of every
file straight into a normalised 16-bit NCHW tensor (training input), encode RGB images to files.
Sizes run from one 64x64 image, where launches and host work are all there is, over single
photographs and small batches, to batches of 67 million pixels.  All three patch sizes of the
format's own rule, ragged and odd sizes, files at any byte alignment, compressible and
incompressible content.

Everything is integer work on bytes (and a table of 16-bit values in the training path), so
outputs are compared exactly and a pass has no floating-point work to speak of.
"""
import math
import random

import torch

import paper_2208_08711_amd as l3

MEAN, STDV = (0.485, 0.456, 0.406), (0.229, 0.224, 0.225)


def _decode(name, images, width, height, patch, **more):
    """width and height are ranges: (least, most) of the images of a batch."""
    case = {"name": name, "op": "decode", "images": images, "width_min": width[0], "width_max": width[1],
            "height_min": height[0], "height_max": height[1], "patch": patch, "content": "scene",
            "layout": "hwc", "align": 64, "prepared": True}
    case.update(more)
    return case


def _train(name, images, width, height, patch, window, dtype, **more):
    case = _decode(name, images, width, height, patch, op="train", window_w=window[0], window_h=window[1],
                   dtype=dtype)
    del case["layout"]
    case.update(more)
    return case


def _encode(name, images, width, height, patch, **more):
    case = _decode(name, images, width, height, patch, op="encode")
    for key in ("layout", "align", "prepared"):
        del case[key]
    case.update(more)
    return case


def listed():
    return [
        # one small image on its own: what a call costs
        _decode("decode_64x64_one", 1, (64, 64), (64, 64), 32, content="smooth", prepared=False),
        # one full-HD frame for a viewer or a serving request, nothing to batch it with
        _decode("decode_fhd_one", 1, (1920, 1920), (1080, 1080), 64, prepared=False),
        # a small per-GPU share of street scenes (large networks train with 1 to 8 of these)
        _decode("decode_street_4", 4, (2048, 2048), (1024, 1024), 128),
        # the headline batch: 32 street scenes
        _decode("decode_street_32", 32, (2048, 2048), (1024, 1024), 128),
        # planar output, as PyTorch wants it; easily compressed content; N = 64
        _decode("decode_fhd_32_planar", 32, (1920, 1920), (1080, 1080), 64, content="smooth_fine", layout="chw"),
        # a classification batch: many small images of all sizes, files end to end in one buffer
        _decode("decode_photos_256", 256, (400, 500), (300, 375), 32, content="smooth", align=1),
        # large frames, half of them incompressible, planar
        _decode("decode_uhd_8_planar", 8, (3840, 3840), (2160, 2160), 128, content="mixed", layout="chw"),
        # training input of a classifier: 224x224 windows with mirror and normalisation, bf16
        _train("train_224_256", 256, (400, 500), (300, 375), 32, (224, 224), "bf16", content="smooth"),
        # training input of a segmentation network: larger windows of street scenes, fp16, arguments
        # made anew for the call as files and windows change from step to step
        _train("train_street_16", 16, (2048, 2048), (1024, 1024), 128, (768, 768), "fp16", prepared=False),
        # one frame encoded as it arrives
        _encode("encode_fhd_one", 1, (1920, 1920), (1080, 1080), 64),
        # data sets written on the GPU: street scenes, and photographs of all sizes
        _encode("encode_street_32", 32, (2048, 2048), (1024, 1024), 128),
        _encode("encode_photos_256", 256, (400, 500), (300, 375), 32, content="smooth"),
    ]


def _log_uniform(rng, least, most):
    return int(round(math.exp(rng.uniform(math.log(least), math.log(most)))))


def draw(rng):
    """One more case: sizes over their whole range, at most 40 million pixels a batch (the
    largest listed ones have 67)."""
    width, height = _log_uniform(rng, 40, 3840), 0
    height = max(24, min(2160, int(width * rng.uniform(0.45, 1.3))))
    spread = rng.choice((1.0, 1.0, 0.7))             # all images of one size, or of several
    low_w, low_h = max(1, int(width * spread)), max(1, int(height * spread))
    total = _log_uniform(rng, width * height, max(40_000_000, width * height))
    images = max(1, min(600, total // (width * height)))
    rule = l3.default_patch(width, height)
    patch = rule if rng.random() < 0.7 else rng.choice((32, 64, 128))
    content = rng.choice(("scene", "scene", "smooth", "smooth_fine", "mixed"))
    sizes = ((low_w, width), (low_h, height), patch)
    op = rng.choice(("decode", "decode", "decode", "train", "encode", "encode"))
    if op == "decode":
        case = _decode("", images, *sizes, content=content, layout=rng.choice(("hwc", "hwc", "chw")),
                       align=rng.choice((1, 64)), prepared=images > 8)
    elif op == "train":
        window = (max(1, int(low_w * rng.uniform(0.4, 1.0))), max(1, int(low_h * rng.uniform(0.4, 1.0))))
        case = _train("", images, *sizes, window, rng.choice(("bf16", "fp16")), content=content,
                      align=rng.choice((1, 64)), prepared=images > 32)
    else:
        case = _encode("", images, *sizes, content=content)
    del case["name"]
    return case


# ---- inputs -----------------------------------------------------------------------------------


def _picture(gen, width, height, content):
    """One uint8 [height, width, 3] image on the GPU."""
    dev = gen.device
    if content == "bytes":
        return torch.randint(0, 256, (height, width, 3), generator=gen, device=dev, dtype=torch.uint8)
    y = torch.arange(height, device=dev, dtype=torch.float32)
    x = torch.arange(width, device=dev, dtype=torch.float32)
    noise = torch.randn((height, width, 3), generator=gen, device=dev)
    if content == "scene":                           # flat regions with dark outlines, and texture
        sites = torch.rand((40, 2), generator=gen, device=dev) * torch.tensor([float(height), float(width)], device=dev)
        colour = torch.rand((40, 3), generator=gen, device=dev) * 255.0
        dist = (y[None, :] - sites[:, :1]).square()[:, :, None] + (x[None, :] - sites[:, 1:]).square()[:, None, :]
        region = dist.argmin(0)
        field = colour[region]
        edge = torch.zeros((height, width), dtype=torch.bool, device=dev)
        edge[:, 1:] |= region[:, 1:] != region[:, :-1]
        edge[1:] |= region[1:] != region[:-1]
        field[edge] = 16.0
        field = field + 3.0 * noise
    else:                                            # a smooth field and sensor noise
        wave = torch.rand((6, 3, 4), generator=gen, device=dev)
        fy = (wave[..., 0] * 0.03).unsqueeze(-1) * y + wave[..., 2:3] * (2 * math.pi)
        fx = (wave[..., 1] * 0.03).unsqueeze(-1) * x
        # cos(a + b) from the two axes' own cosines and sines: [6, 3, height] and [6, 3, width]
        amp = (wave[..., 3:4] * 20.0)
        field = (torch.einsum("kch,kcw->hwc", amp * fy.cos(), fx.cos()) -
                 torch.einsum("kch,kcw->hwc", amp * fy.sin(), fx.sin())) + 128.0
        field = field + (0.93 if content == "smooth_fine" else 6.0) * noise
    return field.round_().clamp_(0, 255).to(torch.uint8)


def _pictures(case, seed):
    """The batch's images, each a view into one buffer.  Their sizes belong to the case (so that
    outputs of two seeds have one shape), what they show to the seed."""
    rng = random.Random(seed * 7919 + 1)
    sizes = random.Random(case["images"] * 65537 + case["width_max"])
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed * 1000003 + 17)
    shapes = [(sizes.randint(case["width_min"], case["width_max"]),
               sizes.randint(case["height_min"], case["height_max"]))
              for _ in range(case["images"])]
    flat = torch.empty(sum(3 * w * h for w, h in shapes), dtype=torch.uint8, device="cuda")
    images, at = [], 0
    for k, (w, h) in enumerate(shapes):
        content = case["content"] if case["content"] != "mixed" else ("smooth", "bytes")[k % 2]
        image = flat[at:at + 3 * w * h].view(h, w, 3)
        image.copy_(_picture(gen, w, h, content))
        images.append(image)
        at += 3 * w * h
    return images, rng


_contexts = {}


def _context():
    """One context a process, as a user's program keeps it."""
    device = torch.cuda.current_device()
    if device not in _contexts:
        _contexts[device] = l3.Context(device)
    return _contexts[device]


def _file_room(images, patch):
    """Room for one file per image in one zeroed buffer (starts 16-byte aligned), the files' views
    and the words for lengths and status."""
    room = [l3.encode_bound(int(im.shape[1]), int(im.shape[0]), patch) for im in images]
    at, starts = 0, []
    for r in room:
        starts.append(at)
        at += (r + 15) // 16 * 16
    buffer = torch.zeros(at, dtype=torch.uint8, device="cuda")
    files = [buffer[s:s + r] for s, r in zip(starts, room)]
    n = len(images)
    return buffer, files, torch.zeros(n, dtype=torch.int64, device="cuda"), torch.zeros(n, dtype=torch.int32, device="cuda")


def _staged_files(images, patch, align):
    """The images' files as a loader would have them: in one buffer on the GPU, one behind the
    other at multiples of `align`, with the headers read on the host."""
    buffer, files, lengths, status = _file_room(images, patch)
    l3.encode_batch(_context(), images, files, lengths, patch=patch, status=status)
    if int(status.abs().sum()):
        raise RuntimeError("an input could not be encoded")
    sizes = lengths.tolist()
    at, starts = 0, []
    for s in sizes:
        starts.append(at)
        at += (s + align - 1) // align * align
    staged = torch.zeros(at + 16, dtype=torch.uint8, device="cuda")
    views = [staged[s:s + n] for s, n in zip(starts, sizes)]
    for view, f, n in zip(views, files, sizes):
        view.copy_(f[:n])
    host = staged.cpu().numpy()
    infos = [l3.peek_header(host[s:s + n]) for s, n in zip(starts, sizes)]
    return views, infos


def prepare(case, seed):
    images, rng = _pictures(case, seed)
    n, patch = case["images"], case["patch"]
    state = {"case": case, "context": _context()}
    if case["op"] == "encode":
        state["images"] = images
        state["buffer"], state["files"], state["lengths"], state["status"] = _file_room(images, patch)
        return state
    files, infos = _staged_files(images, patch, case["align"])
    state["files"], state["infos"] = files, infos
    state["status"] = torch.zeros(n, dtype=torch.int32, device="cuda")
    if case["op"] == "decode":
        planar = case["layout"] == "chw"
        state["layout"] = l3.LAYOUT_CHW if planar else l3.LAYOUT_HWC
        state["pixels"] = torch.zeros(sum(3 * i.width * i.height for i in infos), dtype=torch.uint8, device="cuda")
        state["outs"], at = [], 0
        for i in infos:
            size = 3 * i.width * i.height
            shape = (3, i.height, i.width) if planar else (i.height, i.width, 3)
            state["outs"].append(state["pixels"][at:at + size].view(shape))
            at += size
        if case["prepared"]:
            state["batch"] = l3.PreparedBatch(files, infos, state["outs"], layout=state["layout"])
        return state
    w, h = case["window_w"], case["window_h"]
    state["crops"] = [(rng.randint(0, i.width - w), rng.randint(0, i.height - h), rng.random() < 0.5) for i in infos]
    bf16 = case["dtype"] == "bf16"
    state["dtype"] = l3.BF16 if bf16 else l3.FP16
    state["tensor"] = torch.zeros((n, 3, h, w), dtype=torch.bfloat16 if bf16 else torch.float16, device="cuda")
    if case["prepared"]:
        state["batch"] = l3.PreparedCropBatch(files, infos, state["crops"], MEAN, STDV)
    return state


# ---- one pass ---------------------------------------------------------------------------------


def run(state):
    case = state["case"]
    if case["op"] == "encode":
        l3.encode_batch(state["context"], state["images"], state["files"], state["lengths"], patch=case["patch"],
                        status=state["status"])
        return {"files": state["buffer"], "lengths": state["lengths"], "status": state["status"]}
    if case["op"] == "decode":
        if case["prepared"]:
            l3.decode_batch_prepared(state["context"], state["batch"], status=state["status"])
        else:
            l3.decode_batch(state["context"], state["files"], state["infos"], state["outs"], layout=state["layout"],
                            status=state["status"])
        return {"pixels": state["pixels"], "status": state["status"]}
    w, h = case["window_w"], case["window_h"]
    if case["prepared"]:
        l3.decode_crop_normalize_batch_prepared(state["context"], state["batch"], w, h, state["tensor"],
                                                dtype=state["dtype"], status=state["status"])
    else:
        l3.decode_crop_normalize_batch(state["context"], state["files"], state["infos"], state["crops"], w, h, MEAN,
                                       STDV, state["tensor"], dtype=state["dtype"], status=state["status"])
    return {"tensor": state["tensor"], "status": state["status"]}


# ---- what a pass cannot do without ------------------------------------------------------------

# file bytes per image byte of the generated content (for images of a few patches or more)
_RATIO = {
    "scene": {32: 0.71, 64: 0.75, 128: 0.82},
    "smooth": {32: 0.77, 64: 0.77, 128: 0.76},
    "smooth_fine": {32: 0.44, 64: 0.43, 128: 0.45},
    "mixed": {32: 0.91, 64: 0.90, 128: 0.89},
}


def work(case):
    """Bytes that have to move: files read and pixels written, or the other way round.  A window
    needs the streams of the patches that it touches.  No floating-point work."""
    n, patch = case["images"], case["patch"]
    width = (case["width_min"] + case["width_max"]) / 2
    height = (case["height_min"] + case["height_max"]) / 2
    ratio = _RATIO[case["content"]][patch]
    header = 13 + 12 * math.ceil(width / patch) * math.ceil(height / patch)
    if case["op"] != "train":
        return {"bytes": n * (3 * width * height * (1 + ratio) + header), "flops": 0}
    w, h = case["window_w"], case["window_h"]
    touched = min(width, w + patch - 1) * min(height, h + patch - 1)
    return {"bytes": n * (3 * touched * ratio + header + 6 * w * h), "flops": 0}


def tolerance(case):
    """Lossless: decoded pixels, file bytes and the 16-bit values looked up for them are one
    certain value each."""
    return "exact"
