"""Performance cases of the labeling library: which calls are timed, and on
what inputs.

``listed()`` names the calls that stand for the library's use, ``draw`` gives
further ones over the same ranges, ``prepare`` makes what a program has in
hand before the call (device images, output buffers, a batch context),
``run`` makes the call and ``work`` says what it cannot do without.

Inputs follow ``paper_1708_08180_amd/workloads.py`` (density x grain noise,
smoothed masks, long chains, camera frames, the mixed batch), drawn on the
device where that is quicker.  All outputs are whole numbers.
"""
from __future__ import annotations

import ctypes
import math

import torch

from paper_1708_08180_amd import binding, workloads

COMPONENT_WORDS = binding.COMPONENT_BYTES // 4


def listed():
    return [
        # a region of interest cut from a frame: the smallest calls, where
        # launches and latency count
        {"name": "roi_120x160_c8", "call": "label", "image": "blobs", "H": 120, "W": 160, "conn": 8},
        # one camera frame (moving objects plus salt noise), labeled as it arrives
        {"name": "camera_1080x1920_c8", "call": "label", "image": "blobs", "H": 1080, "W": 1920, "conn": 8},
        # the benchmark's image: independent pixels at p = 0.5
        {"name": "noise_4096x4096_c8", "call": "label", "image": "noise", "H": 4096, "W": 4096, "conn": 8,
         "p": 0.5, "g": 1},
        # a crop of a larger frame: odd sizes and an unaligned row pitch, 4-connectivity
        {"name": "crop_3001x4099_c4", "call": "label", "image": "noise", "H": 3001, "W": 4099, "conn": 4,
         "p": 0.6, "g": 2, "pad": 38},
        # the largest single images: a thresholded smooth field, and one
        # component threaded through every tile
        {"name": "smooth_8192x8192_c8", "call": "label", "image": "smooth", "H": 8192, "W": 8192, "conn": 8,
         "sigma": 4.0},
        {"name": "serpentine_8192x8192_c4", "call": "label", "image": "serpentine", "H": 8192, "W": 8192,
         "conn": 4},
        # a segmentation map: every value class labeled
        {"name": "equal_2160x3840_c8", "call": "equal", "image": "levels", "H": 2160, "W": 3840, "conn": 8,
         "sigma": 5.0, "levels": 6},
        # sizes and places of the objects of a label image
        {"name": "stats_2160x3840", "call": "component_stats", "image": "smooth", "H": 2160, "W": 3840,
         "conn": 8, "sigma": 3.0},
        # labels and statistics in one call, both left on the device for the next stage
        {"name": "label_stats_4096x4096_c8", "call": "label_stats", "image": "noise", "H": 4096, "W": 4096,
         "conn": 8, "p": 0.5, "g": 1},
        # a volume: porous medium, full neighbourhood
        {"name": "volume_256x256x256_c26", "call": "label3d", "image": "noise3d", "D": 256, "H": 256, "W": 256,
         "conn": 26, "p": 0.3},
        # a cut of a scan: odd sizes, face neighbours
        {"name": "volume_97x251x203_c6", "call": "label3d", "image": "smooth3d", "D": 97, "H": 251, "W": 203,
         "conn": 6, "sigma": 2.0},
        # images of five camera resolutions in one call (the batched form)
        {"name": "batch_64_mixed_c8", "call": "batch", "image": "mixed", "n": 64, "sizes_seed": 40000,
         "conn": 8},
    ]


def _log_size(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["label", "label", "label", "equal", "component_stats", "label_stats", "label3d", "batch"])
    conn = rng.choice([4, 8])
    if kind == "batch":
        return {"call": "batch", "image": "mixed", "n": _log_size(rng, 2, 64),
                "sizes_seed": rng.randrange(1, 1 << 30), "conn": conn}
    if kind == "label3d":
        case = {"call": "label3d", "D": _log_size(rng, 16, 256), "H": _log_size(rng, 40, 256),
                "W": _log_size(rng, 40, 256), "conn": rng.choice([6, 18, 26])}
        if rng.random() < 0.5:
            case.update(image="noise3d", p=round(rng.uniform(0.1, 0.5), 3))
        else:
            case.update(image="smooth3d", sigma=round(rng.uniform(1.0, 3.0), 2))
        return case
    case = {"call": kind, "conn": conn}
    hi = 8192 if kind == "label" else 4096
    case["H"], case["W"] = _log_size(rng, 90, hi), _log_size(rng, 90, hi)
    if kind == "equal":
        case.update(image="levels", sigma=round(rng.uniform(2.0, 8.0), 2), levels=rng.randrange(3, 17))
        return case
    image = rng.choice(["blobs", "noise", "smooth"] + (["serpentine"] if kind == "label" else []))
    if image == "blobs":
        case["H"], case["W"] = min(case["H"], 2160), min(case["W"], 3840)
    case["image"] = image
    if image == "noise":
        case.update(p=round(rng.uniform(0.1, 0.9), 3), g=rng.choice([1, 2, 4, 8, 16]))
    elif image == "smooth":
        case["sigma"] = round(rng.uniform(2.0, 8.0), 2)
    if kind == "label":
        case["pad"] = rng.choice([0, 0, rng.randrange(1, 64)])
    return case


# ------------------------------------------------------------------ inputs

def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _blur(z, sigma, axis):
    """Gaussian filter along one axis of a padded field (valid part)."""
    r = int(3.0 * sigma + 0.5)
    w = [math.exp(-0.5 * (k / sigma) ** 2) for k in range(-r, r + 1)]
    n = z.shape[axis] - 2 * r
    out = z.narrow(axis, 0, n) * w[0]
    for k in range(1, 2 * r + 1):
        out.add_(z.narrow(axis, k, n), alpha=w[k])
    return out


def _smooth_field(shape, sigma, gen):
    r = int(3.0 * sigma + 0.5)
    z = torch.randn([s + 2 * r for s in shape], generator=gen, device="cuda", dtype=torch.float32)
    for axis in range(len(shape)):
        z = _blur(z, sigma, axis)
    return z


def _levels(z, levels):
    cut = z.flatten()[:: max(1, z.numel() // 65536)].sort().values
    edges = torch.stack([cut[(k * cut.numel()) // levels] for k in range(1, levels)])
    return torch.bucketize(z, edges).to(torch.uint8)


def _image(case, seed):
    kind = case["image"]
    if kind == "blobs":
        frame = workloads.CameraStream(case["H"], case["W"], int(seed)).step()
        return torch.from_numpy(frame).cuda()
    gen = _generator(seed)
    if kind == "noise3d":
        return (torch.rand((case["D"], case["H"], case["W"]), generator=gen, device="cuda") < case["p"]).to(torch.uint8)
    if kind == "smooth3d":
        return (_smooth_field((case["D"], case["H"], case["W"]), case["sigma"], gen) > 0).to(torch.uint8)
    H, W = case["H"], case["W"]
    if kind == "noise":
        g = case["g"]
        cells = torch.rand((-(-H // g), -(-W // g)), generator=gen, device="cuda") < case["p"]
        cells = cells.to(torch.uint8)
        if g > 1:
            cells = cells.repeat_interleave(g, 0).repeat_interleave(g, 1)[:H, :W]
        return cells.contiguous()
    if kind == "smooth":
        return (_smooth_field((H, W), case["sigma"], gen) > 0).to(torch.uint8)
    if kind == "levels":
        return _levels(_smooth_field((H, W), case["sigma"], gen), case["levels"])
    if kind == "serpentine":
        # full rows joined by one pixel near alternate ends
        img = torch.zeros((H, W), dtype=torch.uint8, device="cuda")
        img[0::2] = 1
        y = torch.arange(1, H, 2, device="cuda")
        off = torch.randint(0, min(64, W), (y.numel(),), generator=gen, device="cuda")
        img[y, torch.where((y // 2) % 2 == 0, W - 1 - off, off)] = 1
        return img
    raise ValueError("unknown image kind %r" % (kind,))


def _padded(img, pad):
    """The image as a view whose rows lie `pad` bytes further apart."""
    if not pad:
        return img
    big = torch.zeros((img.shape[0], img.shape[1] + pad), dtype=torch.uint8, device="cuda")
    big[:, :img.shape[1]] = img
    return big[:, :img.shape[1]]


def _labels_like(img):
    return torch.zeros(tuple(img.shape), dtype=torch.int32, device="cuda")


def prepare(case, seed):
    call = case["call"]
    state = {"call": call, "conn": case["conn"]}
    if call == "batch":
        # the image kinds of the mixed batch, redrawn for every seed
        images = []
        for s in workloads.batch_spec(case["n"], case["sizes_seed"]):
            one = {"H": s.H, "W": s.W}
            if s.kind == "bernoulli":
                one.update(image="noise", p=s.param, g=1)
            else:
                one.update(image="smooth", sigma=s.param)
            images.append(_image(one, seed * 1009 + s.index))
        outs = [_labels_like(im) for im in images]
        ctx = binding.BatchContext(len(images), sum(im.numel() for im in images))
        state.update(images=images, outs=outs, ctx=ctx, descs=ctx.descs(images, outs))
        return state
    img = _padded(_image(case, seed), case.get("pad", 0))
    state["out"] = _labels_like(img)
    state["img"] = img
    if call == "component_stats":
        binding.label(img, case["conn"], out=state["out"])
    if call in ("component_stats", "label_stats"):
        # room for the densest components under the connectivity
        cap = (case["H"] * case["W"]) // (4 if case["conn"] == 8 else 2) + case["H"] + case["W"] + 1
        cap = min(cap, 1 << 21)
        state["records"] = torch.zeros((cap, COMPONENT_WORDS), dtype=torch.int32, device="cuda")
        state["count"] = torch.zeros(1, dtype=torch.int32, device="cuda")
    return state


# -------------------------------------------------------------------- calls

def run(state):
    call, conn = state["call"], state["conn"]
    if call == "label":
        return binding.label(state["img"], conn, out=state["out"])
    if call == "equal":
        return binding.label_equal(state["img"], conn, out=state["out"])
    if call == "label3d":
        return binding.label3d(state["img"], conn, out=state["out"])
    if call == "batch":
        return state["ctx"].label(state["images"], conn, outs=state["outs"], descs=state["descs"])
    # statistics through the C ABI, records left on the device for the next stage
    img, out, rec, cnt = state["img"], state["out"], state["records"], state["count"]
    H, W = img.shape
    lib = binding.load_library()
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    if call == "component_stats":
        rc = lib.ccl_component_stats(out.data_ptr(), H, W, rec.data_ptr(), rec.shape[0], cnt.data_ptr(), stream)
    else:
        rc = lib.ccl_label_2d_stats(img.data_ptr(), H, W, img.stride(0), conn, out.data_ptr(), rec.data_ptr(),
                                    rec.shape[0], cnt.data_ptr(), None, stream)
    if rc != binding.CCL_OK:
        raise RuntimeError("%s failed: status %d" % (call, rc))
    return [rec, cnt] if call == "component_stats" else [out, rec, cnt]


def work(case):
    """Image bytes in and 4-byte labels out once each (statistics of a label
    image: the labels in); the operations are comparisons, none of them
    floating point."""
    if case["call"] == "batch":
        px = sum(s.H * s.W for s in workloads.batch_spec(case["n"], case["sizes_seed"]))
    else:
        px = case.get("D", 1) * case["H"] * case["W"]
    return {"bytes": (4 if case["call"] == "component_stats" else 5) * px, "flops": 0}


def exact(case, seed):
    """Labels and records are whole numbers: there is no nearer value than
    equality."""
    return None
