"""The work that a user of this library has it do, as cases that can be timed.

Every case loads one of the repository's model configurations (synth/configs.py) onto the GPU and sends one batch of
images through one public entry point of `Flow`: `forward` (pixels to latents and prior codes), `inverse` (latents to
pixels), `encode` (pixels to entropy-coded containers), `decode` (containers to pixels), or, for a photograph larger
than the model's own image size, `encode_image` and `decode_image` (patch by patch). All arithmetic is integer, so
every result has to come out the same to the bit.

A program loads a model once and then sees new images: `prepare` keeps one `Flow` per (configuration, batch capacity)
for the life of the process and makes the images (or the latents or containers they give) anew from the seed.
"""
import math

import numpy as np
import torch

import paper_2206_08869_amd as iodf
from synth import CONFIGS, make_blob
from synth.configs import flow_networks, macs_per_image, net_layers

OPS = ("forward", "inverse", "encode", "decode")

# configuration -> (largest batch drawn, weight in the draw)
RANGES = {
    "cfg1": (64, 1),             # tiny two-coupling flow on 8x8 pixels
    "cfg2": (512, 3),            # 32x32, small residual networks at width 128
    "cfg3": (256, 1),            # 32x32, dense networks at width 512
    "cfg4": (128, 1),            # 64x64, dense networks at width 512
    "cfg5": (1024, 1),           # cfg4 with half of the filters gated off
    "paper_res32": (512, 3),     # the paper's own residual networks, 32x32
    "paper_res64": (256, 2),     # ... 64x64
    "paper_iodf64": (256, 2),    # ... pruned
    "paper_iodf64_u": (256, 2),  # ... pruned, unsigned activation codes
    "wide_resnet": (200, 1),     # residual networks 256 wide
    "mid_dense": (256, 1),       # dense networks 256 wide
    "odd_dense_g": (512, 1),     # 45 kept channels: a multiple of nothing
    "rect_resnet_g": (256, 1),   # 24x40 images, gated residual networks
}
IMAGE_MODELS = ("paper_res64", "paper_iodf64", "paper_iodf64_u")


def listed():
    def case(name, model, op, batch, **more):
        return dict(name=name, model=model, op=op, batch=batch, **more)
    return [
        # the smallest call: one tiny image, a handful of launches
        case("tiny_forward_1", "cfg1", "forward", 1),
        # a training-set-sized batch of small images through the small residual flow
        case("resnet32_forward_64", "cfg2", "forward", 64),
        # an odd batch of 32x32 images to containers with the paper's own network (a data loader's last batch)
        case("paper32_encode_37", "paper_res32", "encode", 37),
        # one 64x64 image at a time, decoded as it arrives (the paper's latency case, its own pruned network)
        case("paper64p_decode_1", "paper_iodf64", "decode", 1),
        # bulk compression of 64x64 images with the paper's own network
        case("paper64_encode_256", "paper_res64", "encode", 256),
        # bulk decompression with the pruned network in the paper's unsigned format
        case("paper64pu_decode_256", "paper_iodf64_u", "decode", 256),
        # a photograph coded in 64x64 patches, sides that are no multiples of 64, several sub-batches
        case("photo_encode", "paper_iodf64", "encode_image", 64, h=600, w=1000),
        # the dense 32x32 flow on an odd batch, decode direction
        case("dense32_inverse_50", "cfg3", "inverse", 50),
        # the headline workload: dense 64x64 flow, encode and decode directions
        case("dense64_forward_128", "cfg4", "forward", 128),
        case("dense64_inverse_128", "cfg4", "inverse", 128),
        # latency of one image through the gate-pruned dense flow
        case("pruned64_forward_1", "cfg5", "forward", 1),
        # throughput of the gate-pruned dense flow at its largest batch
        case("pruned64_forward_1024", "cfg5", "forward", 1024),
    ]


def draw(rng):
    names = sorted(RANGES)
    model = rng.choices(names, [RANGES[n][1] for n in names])[0]
    if model in IMAGE_MODELS and rng.random() < 0.25:
        return dict(model=model, op=rng.choice(("encode_image", "decode_image")), batch=rng.choice((32, 64, 100)),
                    h=rng.randint(65, 900), w=rng.randint(65, 900))
    top = RANGES[model][0]
    batch = min(top, max(1, int(round(math.exp(rng.uniform(0.0, math.log(top + 0.49)))))))
    return dict(model=model, op=rng.choice(OPS), batch=batch)


_blobs, _flows = {}, {}


def _flow(model, capacity):
    """The loaded model, kept as a program keeps it."""
    key = (model, capacity)
    if key not in _flows:
        if model not in _blobs:
            _blobs.clear()  # the dense models are 1 GB of host memory each
            _blobs[model] = make_blob(CONFIGS[model])
        _flows[key] = iodf.Flow(_blobs[model], max_batch=capacity, device=0)
    return _flows[key]


def _images(n, h, w, kind, seed):
    """uint8 [n,3,h,w]: white noise blurred with a Gaussian of 2 px, mean 128 and deviation 50 (as synth/images.py), or uniform bytes."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    if kind == "uniform":
        return torch.randint(0, 256, (n, 3, h, w), generator=gen, device="cuda", dtype=torch.uint8)
    g = torch.randn((n, 3, h, w), generator=gen, device="cuda")
    taps = np.exp(-0.5 * (np.arange(-6, 7) / 2.0) ** 2)
    for dim in (2, 3):
        g = sum(float(k) * torch.roll(g, i - 6, dims=dim) for i, k in enumerate(taps / taps.sum()))
    g = g - g.mean(dim=(1, 2, 3), keepdim=True)
    g = g / g.std(dim=(1, 2, 3), keepdim=True) * 50.0 + 128.0
    return g.round().clamp_(0, 255).to(torch.uint8).contiguous()


def prepare(case, seed):
    cfg = CONFIGS[case["model"]]
    op, b = case["op"], case["batch"]
    flow = _flow(case["model"], b)
    state = dict(op=op, flow=flow)
    if op in ("encode_image", "decode_image"):
        img = _images(1, case["h"], case["w"], cfg.image_kind, seed)[0].contiguous()
        state.update(h=case["h"], w=case["w"])
        if op == "encode_image":
            state["img"] = img
        else:
            state["parts"] = flow.encode_image(img)
        return state
    x = _images(b, cfg.H, cfg.W, cfg.image_kind, seed)
    if op in ("forward", "encode"):
        state["x"] = x
    elif op == "inverse":
        state["z"] = flow.forward(x, want_codes=False)[0]
    else:
        state["words"] = flow.encode(x)[0]
    return state


def run(state):
    flow, op = state["flow"], state["op"]
    if op == "forward":
        return flow.forward(state["x"])
    if op == "inverse":
        return flow.inverse(state["z"])
    if op == "encode":
        return flow.encode(state["x"])
    if op == "decode":
        return flow.decode(state["words"])
    if op == "encode_image":
        return flow.encode_image(state["img"])
    return flow.decode_image(state["parts"], state["h"], state["w"])


def _weight_bytes(cfg, with_heads):
    """Kept weights and constants of every network that runs, read once."""
    total = 0
    for kind, lv, _c, c_in, c_out in flow_networks(cfg):
        if kind == 1 and not with_heads:
            continue
        keep = cfg.keep_at(lv)
        wk = max(1, int(round(cfg.width * keep))) if keep < 1.0 else cfg.width
        for i, (co, ci, k, _relu, _sc, gated) in enumerate(
                net_layers(cfg.family, c_in, c_out, cfg.width, cfg.depth, cfg.block_k2)):
            rows = wk if gated else co
            total += rows * (ci if i == 0 else ci // cfg.width * wk) * k * k + 9 * rows
    return total


def work(case):
    cfg = CONFIGS[case["model"]]
    op, n = case["op"], case["batch"]
    if op in ("encode_image", "decode_image"):
        n = -(-case["h"] // cfg.H) * -(-case["w"] // cfg.W)
    heads = cfg.heads and op != "inverse"
    if op in ("forward", "inverse"):
        per_image = cfg.d * 5 + (cfg.d_codes if op == "forward" else 0)  # pixels, int32 latents, codes
    else:
        per_image = cfg.d * 3                                            # pixels, and about 16 bits of container a value
    return {"bytes": n * per_image + _weight_bytes(cfg, heads), "flops": 2 * n * macs_per_image(cfg, with_heads=heads)}


def tolerance(case):
    return "exact"
