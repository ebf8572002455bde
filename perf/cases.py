"""Workloads of the activation codec: what a training or inference program has it do.

A case is one pass through the public entry points of ``paper_2111_09562_amd``: a compression after a
layer's forward pass, a decompression for its backward pass, both for a set of layers on streams of their
own, or the saved-tensor hook around a small differentiable layer.  Inputs are seeded synthetic activations
made on the GPU with the statistics of post-ReLU feature maps: smoothed Gaussian fields, standardised per
channel, shifted, rectified (about half zeros); or a rectified Laplace field without any smoothness.
"""
from __future__ import annotations

import math

import torch
import torch.nn.functional as F

from paper_2111_09562_amd import comet
from paper_2111_09562_amd.autograd import saved_activations

# Bits of a container per element for (error bound, smoothness): what the codec needs at these bounds on
# such fields, log-linear between the entries.
_RATE = {"blur": ((1e-4, 11.9), (1e-3, 9.2), (1e-2, 6.7), (1e-1, 3.95)), "laplace": ((1e-4, 15.0), (1e-3, 12.1), (1e-2, 8.9), (1e-1, 5.7))}


def _case(name, op, shape, eb, nbins, dtype="float32", field="blur", blur=3, shift=-0.2, chunk=64, zero_chunks=False, sync=False, static=False):
    n, c, h, w = shape
    return dict(name=name, op=op, n=n, c=c, h=h, w=w, eb=eb, nbins=nbins, dtype=dtype, field=field, blur=blur, shift=shift,
                chunk=chunk, zero_chunks=zero_chunks, sync=sync, static=static)


def listed():
    return [
        # One image through a late layer, compressed when its size is needed at once (exact-size buffers).
        _case("compress_one_image", "compress", (1, 64, 28, 28), 1e-2, 1024, sync=True),
        # The same size brought back from a serving loop that holds no context and allocates nothing.
        _case("decompress_one_image", "decompress", (1, 64, 28, 28), 1e-2, 1024, static=True),
        # A layer of a small batch in a training step under the saved-tensor hook: forward packs, backward unpacks.
        _case("hook_training_layer", "hook", (8, 64, 56, 56), 1e-2, 1024, sync=True),
        # The first feature map of an image classifier at batch 64, after its forward pass.
        _case("compress_112", "compress", (64, 64, 112, 112), 1e-2, 1024),
        # The layer behind it under a tighter bound (escaped residuals in most rows), for its backward pass.
        _case("decompress_56_tight", "decompress", (64, 256, 56, 56), 1e-3, 1024),
        # Mixed precision with odd planes (no pairs of columns): bfloat16 forward ...
        _case("compress_bf16_odd", "compress", (48, 192, 27, 27), 1e-2, 1024, dtype="bfloat16"),
        # ... and backward.
        _case("decompress_bf16_odd", "decompress", (96, 96, 55, 55), 1e-2, 1024, dtype="bfloat16"),
        # A whole training step's activations: five layers compressed in forward order and brought back in reverse,
        # one context and stream per layer.
        _case("step_five_layers", "step", (64, 64, 112, 112), 1e-2, 1024),
        # A very fine bound: an alphabet of tens of thousands of symbols.
        _case("compress_56_finest", "compress", (64, 256, 56, 56), 1e-4, 65536, shift=0.0),
        # The largest tensor of a wide network at batch 128, heavy-tailed and rough, large alphabet.
        _case("decompress_224_heavy_tail", "decompress", (128, 64, 224, 224), 1e-3, 65536, field="laplace"),
        # Between two refreshes of a layer's statistics: compressed with the code book of its last compression.
        _case("recompress_56_given_book", "given", (64, 256, 56, 56), 1e-2, 1024),
        # Wide planes (dense prediction on whole images): there and back.
        _case("roundtrip_wide_planes", "roundtrip", (2, 16, 480, 854), 1e-2, 1024, sync=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["compress", "compress", "decompress", "decompress", "roundtrip", "given", "hook", "step"])
    elems = math.exp(rng.uniform(math.log(5e4), math.log(6e7)))          # elements of the tensor, of the first layer of a set
    if op == "step":
        side = rng.choice([32, 48, 64, 96, 112])
        n = max(1, round(elems / (64 * side * side)))
        shape = (n, 64, side, side)
    else:
        wide = op in ("compress", "decompress", "roundtrip") and rng.random() < 0.12
        w = _log_int(rng, 513, 2048) if wide else _log_int(rng, 4, 320)
        h = max(1, round(w * rng.uniform(0.6, 1.0)))
        planes = max(1, round(elems / (h * w)))
        c = min(planes, rng.choice([16, 24, 64, 96, 192, 256, 512, 1000]))
        n = max(1, round(planes / c))
        shape = (n, c, h, w)
    n_el = shape[0] * shape[1] * shape[2] * shape[3]
    eb, nbins = rng.choice([(1e-2, 1024), (1e-2, 1024), (1e-3, 1024), (5e-2, 256), (1e-2, 4096), (3e-3, 4096), (1e-3, 16384), (1e-3, 65536), (1e-4, 65536)])
    field = "laplace" if nbins == 65536 and rng.random() < 0.5 else "blur"
    dtype = rng.choice(["float32", "float32", "bfloat16", "float16"])
    if shape[3] > 512 or op in ("given", "step"):
        dtype = "float32"
    if (op in ("given", "step") and nbins > 8192) or (op == "step" and eb / nbins < 5e-7):    # (a set has layers at a tenth of the bound)
        eb, nbins = 1e-2, 1024
    case = _case("", op, shape, eb, nbins, dtype=dtype, field=field, blur=rng.choice([3, 5]), shift=rng.choice([-0.2, 0.0]),
                 chunk=rng.choice([64, 64, 64, 64, 128, 256]), zero_chunks=rng.random() < 0.2, sync=rng.random() < 0.5,
                 static=op == "decompress" and dtype == "float32" and n_el <= comet.STATIC_MAX_ELEMS and rng.random() < 0.3)
    if op == "hook":
        case["sync"] = True
    del case["name"]
    return case


def _shape(case):
    return case["n"], case["c"], case["h"], case["w"]


def _layers(case):
    """(shape, error bound) of every tensor of a case: one, or a set of five whose planes halve while their number grows."""
    n, c, h, w = _shape(case)
    if case["op"] != "step":
        return [((n, c, h, w), case["eb"])]
    chans, bounds = (1, 4, 8, 16, 32), (1.0, 0.1, 5.0, 1.0, 0.1)
    return [((n, c * m, max(1, h >> i), max(1, w >> i)), case["eb"] * b) for i, (m, b) in enumerate(zip(chans, bounds))]


def _activation(case, shape, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    if case["field"] == "laplace":
        x = torch.empty(shape, device="cuda").exponential_(generator=g)
        for part in x.split(max(1, shape[0] // 8)):
            part.mul_(torch.rand(part.shape, device="cuda", generator=g) < 0.5)
    else:
        x = torch.randn(shape, device="cuda", generator=g)
        for part in x.split(max(1, shape[0] // 8)):
            part.copy_(F.avg_pool2d(part, case["blur"], stride=1, padding=case["blur"] // 2))
        std, mean = torch.std_mean(x, dim=(0, 2, 3), keepdim=True, correction=0)
        x.sub_(mean).div_(std.clamp_min(1e-6)).add_(case["shift"]).clamp_min_(0.0)
    return x.to(getattr(torch, case["dtype"]))


def _buffer(shape):
    """A container buffer: a good four fifths of the fp32 size, the worst case for tensors so small that it is cheap."""
    n = shape[0] * shape[1] * shape[2] * shape[3]
    return torch.zeros((int(3.4 * n) + (1 << 20)) // 16 * 16, dtype=torch.uint8, device="cuda")


class _Tensor:
    """One activation with everything the calls on it take."""

    def __init__(self, case, shape, eb, seed):
        self.shape, self.eb = shape, eb
        self.x = _activation(case, shape, seed)
        self.fp32 = self.x.dtype == torch.float32
        self.ctx = comet.Context(self.x.numel(), case["nbins"])
        self.ctx.comet_set_chunk_syms(case["chunk"])
        self.ctx.comet_set_zero_chunks(case["zero_chunks"])
        self.box = _buffer(shape)
        self.out = torch.empty_like(self.x)
        self.stream = None

    def compress(self, nbins, sync):
        f = self.ctx.comet_compress if self.fp32 else self.ctx.comet_compress_16
        return f(self.x, self.eb, nbins, self.box, stream=self.stream, sync=sync)

    def decompress(self, used):
        f = self.ctx.comet_decompress if self.fp32 else self.ctx.comet_decompress_16
        f(self.box, used, self.shape, self.out, stream=self.stream)


def prepare(case, seed):
    ts = [_Tensor(case, shape, eb, seed * 8 + i) for i, (shape, eb) in enumerate(_layers(case))]
    state = {"case": case, "tensors": ts}
    t = ts[0]
    if case["op"] in ("decompress", "given"):
        state["used"] = t.compress(case["nbins"], True)
        if case["op"] == "given":
            state["book"] = t.box[comet.HEADER_BYTES:comet.HEADER_BYTES + case["nbins"]].clone()
        else:
            t.x = None
    elif case["op"] == "hook":
        state["grad"] = torch.randn(t.shape, device="cuda", generator=torch.Generator(device="cuda").manual_seed(seed * 8 + 7)).to(t.x.dtype)
        t.x.requires_grad_(True)
    elif case["op"] == "step":
        for u in ts:
            u.stream = torch.cuda.Stream()
    return state


def run(state):
    case, t = state["case"], state["tensors"][0]
    op, nbins = case["op"], case["nbins"]
    if op == "compress":
        t.compress(nbins, case["sync"])
        return t.box                                         # (behind the container the buffer is zero, as it was made)
    if op == "given":
        t.ctx.comet_compress_with_codebook(t.x, t.eb, nbins, state["book"], t.box, sync=case["sync"])
        return t.box
    if op == "decompress":
        if case["static"]:
            comet.comet_decompress_static(t.box, state["used"], t.shape, t.out)
        else:
            t.decompress(state["used"])
        return t.out
    if op == "roundtrip":
        used = t.compress(nbins, case["sync"])
        t.decompress(used if case["sync"] else t.box.numel())
        return t.box, t.out
    if op == "hook":
        with saved_activations(t.ctx, t.eb, nbins, min_elems=1 << 15, capacity_frac=0.9):
            y = F.silu(t.x)
        (g,) = torch.autograd.grad(y, t.x, state["grad"])
        return y.detach(), g
    here = torch.cuda.current_stream()
    for u in state["tensors"]:
        u.stream.wait_stream(here)
        u.compress(nbins, False)
    for u in reversed(state["tensors"]):
        u.decompress(u.box.numel())
        here.wait_stream(u.stream)
    return [u.out for u in state["tensors"]]


def work(case):
    """Input read once, output written once; about a multiplication and an addition per element each way."""
    total = flops = 0
    for (n, c, h, w), eb in _layers(case):
        el = n * c * h * w
        tensor = el * (4 if case["dtype"] == "float32" else 2)
        pts = _RATE[case["field"]]
        x = min(max(math.log10(eb), -4.0), -1.0)
        k = min(int(x + 4.0), 2)
        box = el * (pts[k][1] + (pts[k + 1][1] - pts[k][1]) * (x + 4.0 - k)) / 8
        once = tensor + box
        if case["op"] == "hook":                             # forward: x, y, container; backward: container, gradient in and out
            total += 4 * tensor + 2 * box
        else:
            total += once * (2 if case["op"] in ("step", "roundtrip") else 1)
        flops += el * (4 if case["op"] in ("step", "roundtrip", "hook") else 2)
    return {"bytes": int(total), "flops": int(flops)}


def tolerance(case):
    # Containers are bytes and every float step of the codec is one correctly rounded operation, so the values
    # that come back are fixed to the last bit; the hook's layer is elementwise.
    return "exact"
