"""The calls this library is timed on: training steps, inference and the image data-flow, through the Python binding.

A case is a plain dict.  `call` says what a pass is:

  step       SeqTrainer.step on one batch of fp32 images (or feature maps), gradients asked for
  encoded    SeqTrainer.step_encoded: the same on a batch that arrives as encoded 8-bit images
  predict    SeqTrainer.predict: logits with the running BatchNorm statistics
  dataflow   encode of a set of 8-bit images, then the decode layer (normalised, cast to the storage type)
  lossless   encode_lossless, then decode_lossless

`net` is a list of units separated by blanks: cN = 3x3 conv + BatchNorm + ReLU to N channels, rN = 3x3 conv + bias + ReLU,
bN = basic block, nN = bottleneck block (N output channels), p = 2x2 max-pool, "/2" behind a unit = stride 2, and last
the head: gap or flat.  The networks are the benchmark configurations of this repository (workloads.config) or a run of
neighbouring units of one: a training step in 16-bit storage amplifies one different rounding by about 1.4 per unit, so
only short runs of units can be compared between two correct implementations.
"""
import math

import torch

from paper_2105_00619_amd import binding as B
from paper_2105_00619_amd import workloads as W

PRECISION = {"fp32": W.FP32, "bf16": W.BF16, "fp16": W.FP16}
DTYPE = {"fp32": torch.float32, "bf16": torch.bfloat16, "fp16": torch.float16}
VGG11 = "c64 p c128 p c256 c256 p c512 c512 p c512 c512 p flat"
RESNET18 = "c64 b64 b64 b128/2 b128 b256/2 b256 b512/2 b512 gap"
RESNET50 = "c64 n256 n256 n256 n512/2 n512 n512 n512 n1024/2 n1024 n1024 n1024 n1024 n1024 n2048/2 n2048 n2048 gap"


def _net(name, call, net, batch, size, precision, width=0, channels=3, classes=100, k=2, momentum=0.0, z=0):
    c = {"call": call, "net": net, "batch": batch, "height": size, "width": width or size, "channels": channels,
         "classes": classes, "precision": precision, "k": k, "momentum": momentum, "z": z}
    return {"name": name, **c} if name else c


def _images(name, call, images, size, channels, z, precision="bf16"):
    c = {"call": call, "batch": images, "height": size, "width": size, "channels": channels, "z": z, "precision": precision}
    return {"name": name, **c} if name else c


def listed():
    return [
        # the smallest training step (workloads.config(1)): a few dozen short kernels, launches and latency
        _net("step_tiny_fp32", "step", "r8 r8 gap", 8, 32, "fp32", classes=10),
        # VGG-11 with BatchNorm in fp32 at an ordinary batch (workloads.config(2)), the whole network
        _net("step_vgg11_fp32", "step", VGG11, 128, 32, "fp32", classes=10, k=4),
        # large images, few of them, fp32: first stages of ResNet-18 at 512 x 512 (workloads.config(6))
        _net("step_basic_fp32_512px", "step", "c64 b64 b128/2 gap", 4, 512, "fp32", classes=10),
        # ResNet-18 training in bf16 with momentum (workloads.config(3)): its first two stages on images
        _net("step_basic_early_bf16", "step", "c64 b64 b128/2 gap", 256, 32, "bf16", momentum=0.9),
        # ... and its last ones, trained on the feature maps that enter them
        _net("step_basic_late_fp16", "step", "b256 b512/2 gap", 256, 8, "fp16", channels=256, momentum=0.9),
        # ResNet-50 training in fp16 with a loss scale (workloads.config(4)): its first stages on images
        _net("step_bottleneck_early_fp16", "step", "c64 n256 n256 n512/2 gap", 512, 32, "fp16"),
        # the stage that carries most of the 152-layer network's step (workloads.config(5)): 8 x 8 maps, batch 4096
        _net("step_bottleneck_mid_bf16", "step", "n1024 n1024 gap", 4096, 8, "bf16", channels=1024),
        # the same network's first stage: the largest activations (4 M pixels)
        _net("step_bottleneck_wide_bf16", "step", "c64 n256 n256 gap", 4096, 32, "bf16"),
        # a batch of odd-sized images that arrives encoded, a ragged last group, pools on odd maps
        _net("step_encoded_odd_fp16", "encoded", "c64 p b128 p b256/2 gap", 99, 45, "fp16", width=37, classes=10, z=7),
        # evaluation of a whole network at the batch it trains with
        _net("predict_resnet50_fp16", "predict", RESNET50, 512, 32, "fp16", k=8),
        # inference on a few images (the batch of the paper's experiments): latency
        _net("predict_resnet18_b16_fp16", "predict", RESNET18, 16, 32, "fp16", k=4),
        # a training set of 8-bit images encoded, then unpacked by the decode layer
        _images("dataflow_50000_bf16", "dataflow", 50000, 32, 3, 16),
    ]


# ---- drawn cases -----------------------------------------------------------------------------------------------------

def _log_uniform(rng, lo, hi):
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return max(lo, min(hi, v))


def _block_run(rng, precision):
    """A run of neighbouring units, the channels that enter it and a range of map sizes in which it occurs."""
    kind = rng.choice(["basic", "bottleneck", "plain"])
    if kind == "plain":  # the VGG widths
        w = rng.choice([64, 128, 256])
        return "c%d p c%d p flat" % (w, 2 * w), 3, (16, 48)
    first = rng.choice([64, 128, 256] if kind == "basic" else [256, 512, 1024])
    letter = "b" if kind == "basic" else "n"
    units = ["%s%d" % (letter, first)]
    if precision != "bf16" and rng.random() < 0.3:
        units *= 2
    if rng.random() < 0.5:
        units.append("%s%d/2" % (letter, 2 * first))
    if first == (64 if kind == "basic" else 256):
        return " ".join(["c64"] + units + ["gap"]), 3, (24, 64)
    return " ".join(units + ["gap"]), first, ((12, 36) if first in (128, 512) else (7, 20))


def draw(rng):
    call = rng.choice(["step", "step", "step", "predict", "encoded", "dataflow", "lossless"])
    if call in ("dataflow", "lossless"):
        size = _log_uniform(rng, 8, 224)
        channels = rng.choice([1, 3, 3, 4])
        most = 150_000_000 // (size * size * channels)
        return _images("", call, _log_uniform(rng, 16, max(17, min(50000, most))), size, channels,
                       rng.randint(1, 16 if call == "dataflow" else 32), rng.choice(["fp32", "bf16", "fp16"]))
    precision = rng.choice(["fp32", "bf16", "bf16", "fp16"])
    net, channels, (lo, hi) = _block_run(rng, precision)
    if call == "encoded" and channels != 3:
        call = "step"
    if call == "predict" and rng.random() < 0.5:
        net, channels, lo, hi = rng.choice([RESNET18, "c64 n256 n512/2 n1024/2 n2048/2 gap"]), 3, 24, 64
    size = rng.randint(lo, hi)
    width = size if rng.random() < 0.6 else rng.randint(lo, hi)
    c = _net("", call, net, 1, size, precision, width=width, channels=channels, classes=rng.choice([10, 100]),
             k=rng.choice([1, 2, 3]), momentum=rng.choice([0.0, 0.9]), z=rng.randint(1, 16) if call == "encoded" else 0)
    # the batch: over the range that costs at most about a third of the largest listed case
    w = work(c)
    cost = w["flops"] / (60e12 if precision == "fp32" else 400e12) + w["bytes"] / 2.5e12
    lo_batch, hi_batch = 1 if call == "predict" else 16, min(4096, int(0.010 / cost))
    c["batch"] = _log_uniform(rng, lo_batch, max(lo_batch + 1, hi_batch))
    if "n" in net.split()[-2]:  # bottleneck networks: the multiples of 32 that they are trained and evaluated with
        c["batch"] = max(32, c["batch"] // 32 * 32)
    return c


# ---- the network a case describes ------------------------------------------------------------------------------------

def _parse(case):
    """[(letter, channels out, stride)] of the body and the head's name."""
    words = case["net"].split()
    body = []
    for t in words[:-1]:
        t, _, s = t.partition("/")
        body.append((t[0], int(t[1:] or 0), int(s or 1)))
    return body, words[-1]


def _units(case):
    body, head = _parse(case)
    c, h, w = case["channels"], case["height"], case["width"]
    units = []
    for letter, n, s in body:
        if letter == "p":
            units.append(W.maxpool())
            h, w = h // 2, w // 2
            continue
        if letter in "cr":
            units.append(W.conv(c, n, stride=s, bn=letter == "c"))
        else:
            units.append((W.basic_block if letter == "b" else W.bottleneck)(c, n, s))
        c, h, w = n, (h - 1) // s + 1, (w - 1) // s + 1
    units.append(W.gap_linear_ce(c, case["classes"]) if head == "gap" else W.flatten_linear_ce(c, case["classes"]))
    return units


def _layers(case):
    """Every convolution and linear layer as (unit, kind, cin, cout, ksize, stride, h, w, bn), with the map it reads, in the
    order of the flat parameter vector: unit order, inside a block conv1, conv2, [conv3], then the projection shortcut."""
    body, head = _parse(case)
    c, h, w = case["channels"], case["height"], case["width"]
    out = []
    for u, (letter, n, s) in enumerate(body):
        if letter == "p":
            h, w = h // 2, w // 2
            continue
        p, q = (h - 1) // s + 1, (w - 1) // s + 1
        if letter in "cr":
            out.append((u, "conv", c, n, 3, s, h, w, letter == "c"))
        else:
            if letter == "b":
                out += [(u, "conv", c, n, 3, s, h, w, True), (u, "conv", n, n, 3, 1, p, q, True)]
            else:
                m = n // 4
                out += [(u, "conv", c, m, 1, 1, h, w, True), (u, "conv", m, m, 3, s, h, w, True),
                        (u, "conv", m, n, 1, 1, p, q, True)]
            if c != n or s != 1:
                out.append((u, "shortcut", c, n, 1, s, h, w, True))
        c, h, w = n, p, q
    out.append((len(body), "linear", c if head == "gap" else c * h * w, case["classes"], 1, 1, 1, 1, False))
    return out


def _params(case, gen):
    """He-normal weights; BatchNorm scales around 1 and shifts around 0 as in a network that has trained for a while."""
    parts = []

    def normal(n, std, mean=0.0):
        parts.append(torch.randn(n, generator=gen, device="cuda") * std + mean)

    for _, kind, cin, cout, k, _, _, _, bn in _layers(case):
        normal(cout * k * k * cin, math.sqrt((1.0 if kind == "linear" else 2.0) / (k * k * cin)))
        if bn:
            normal(cout, 0.2, 1.0)
            normal(cout, 0.1)
        else:
            normal(cout, 0.1)
    return torch.cat(parts)


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 1000003 + 17)


def _input(case, gen):
    """Images: per-channel Gaussians clipped to [0, 1].  Feature maps: what a ReLU gives, half of the values zero."""
    shape = (case["batch"], case["height"], case["width"], case["channels"])
    x = torch.randn(shape, generator=gen, device="cuda")
    return x.mul_(0.25).add_(0.5).clamp_(0.0, 1.0) if case["channels"] <= 4 else x.clamp_(min=0.0)


def _pixels(case, gen):
    shape = (case["batch"], case["height"], case["width"], case["channels"])
    x = torch.randn(shape, generator=gen, device="cuda")
    return x.mul_(64.0).add_(128.0).clamp_(0.0, 255.0).round_().to(torch.uint8)


def _normalisation(case):
    """(scale, shift) per channel of the decode layer: pixel / 255, mean 0.5, deviation 0.25."""
    return [1.0 / (255.0 * 0.25)] * case["channels"], [-2.0] * case["channels"]


def _inputs(case, seed):
    gen = _generator(seed)
    if case["call"] in ("dataflow", "lossless"):
        return {"pixels": _pixels(case, gen)}
    d = {"params": _params(case, gen),
         "y": torch.randint(0, case["classes"], (case["batch"],), generator=gen, device="cuda", dtype=torch.int32)}
    if case["call"] == "encoded":
        d["pixels"] = _pixels(case, gen)
    else:
        d["x"] = _input(case, gen)
    if case["call"] == "predict":
        d["seen"] = _input(case, gen)  # the batch whose statistics the running estimates hold
    return d


# ---- a pass ----------------------------------------------------------------------------------------------------------

LR = 1e-4


def prepare(case, seed):
    d = _inputs(case, seed)
    s = {"case": case}
    if case["call"] in ("dataflow", "lossless"):
        s["pixels"] = d["pixels"]
        if case["call"] == "dataflow":
            groups, n_pos = -(-case["batch"] // case["z"]), case["height"] * case["width"] * case["channels"]
            s["words"] = torch.empty((groups, n_pos, B.encoded_words(case["z"])), dtype=torch.int64, device="cuda")
            s["decoded"] = torch.empty((case["batch"], n_pos), dtype=DTYPE[case["precision"]], device="cuda")
        return s
    predict = case["call"] == "predict"
    t = B.SeqTrainer(_units(case), k_segments=min(case["k"], len(case["net"].split())), plan_mode=2,
                     precision=PRECISION[case["precision"]], batch=case["batch"], height=case["height"], width=case["width"],
                     channels=case["channels"], num_classes=case["classes"], momentum=case["momentum"],
                     bn_momentum=1.0 if predict else 0.0,
                     loss_scale_init=1024.0 if case["precision"] == "fp16" else 0.0)
    t.set_params(d["params"])
    s["trainer"] = t
    if predict:
        s["x"] = d["x"]
        t.step(d["seen"], d["y"], 0.0)  # running statistics of a batch; the weights stay
        return s
    s["y"] = d["y"]
    s["grads"] = torch.empty(t.param_count, dtype=torch.float32, device="cuda")
    if case["call"] == "encoded":
        s["a"] = B.encode(d["pixels"], case["z"])
        s["scale"], s["shift"] = _normalisation(case)
    else:
        s["x"] = d["x"]
    return s


def run(s):
    case = s["case"]
    call = case["call"]
    if call == "step":
        r = s["trainer"].step(s["x"], s["y"], LR, grads=s["grads"])
        return {"loss": r["loss"], "grads": s["grads"]}
    if call == "encoded":
        r = s["trainer"].step_encoded(s["a"], case["z"], s["scale"], s["shift"], s["y"], LR, grads=s["grads"])
        return {"loss": r["loss"], "grads": s["grads"]}
    if call == "predict":
        return {"logits": s["trainer"].predict(s["x"])}
    n_pos = case["height"] * case["width"] * case["channels"]
    if call == "dataflow":
        scale, shift = _normalisation(case)
        B.encode(s["pixels"], case["z"], out=s["words"])
        B.decode_normalized(s["words"], case["batch"], n_pos, case["z"], case["channels"], scale, shift,
                            PRECISION[case["precision"]], out=s["decoded"])
        return {"words": s["words"], "decoded": s["decoded"]}
    a, o = B.encode_lossless(s["pixels"], case["z"])
    return {"words": a, "parity": o, "pixels": B.decode_lossless(a, o, case["batch"], n_pos, case["z"])}


def work(case):
    """Arithmetic: the convolutions and the linear layer, once for a forward pass and three times for a training step (the
    first layer has no data gradient).  Bytes: inputs, parameters and results, and the tensors between layers, which no
    cache holds at the larger sizes: a convolution's output is written and read once in a forward pass; a training step
    reads it once more in its backward pass and writes and reads its gradient."""
    e = 4 if case["precision"] == "fp32" else 2
    n = case["batch"]
    if case["call"] in ("dataflow", "lossless"):
        pos = case["height"] * case["width"] * case["channels"]
        groups = -(-n // case["z"])
        if case["call"] == "dataflow":  # pixels read, words written, words read, decoded values written
            return {"bytes": n * pos * (1 + e) + 2 * groups * pos * 8 * (-(-case["z"] // 8)), "flops": 0}
        return {"bytes": n * pos * 2 + 2 * groups * pos * (8 * (-(-7 * case["z"] // 64)) + 4), "flops": 0}
    train = case["call"] != "predict"
    flops = weights = between = 0
    for i, (_, kind, cin, cout, k, s, h, w, _) in enumerate(_layers(case)):
        p, q = (h - 1) // s + 1, (w - 1) // s + 1
        f = 2 * n * p * q * cout * cin * k * k
        flops += f * ((2 if i == 0 else 3) if train else 1)
        weights += cout * cin * k * k
        between += n * p * q * cout * e
    pixels = n * case["height"] * case["width"] * case["channels"] * (1 if case["call"] == "encoded" else 4)
    if train:  # fp32 weights read and written, gradients written
        return {"bytes": pixels + 12 * weights + 5 * between, "flops": flops}
    return {"bytes": pixels + e * weights + 2 * between + 4 * n * case["classes"], "flops": flops}


def tolerance(case):
    """Sums in another order (the batch permuted) move the gradients of these networks by up to 1e-6 in fp32 where no ReLU
    decision changes and by 1e-3 where one does (the distance to 64 bits shows it), by up to 6e-3 in 16 bits, the
    logits of 50 layers in fp16 by 9e-3; four times that is allowed, but no more than 3e-2."""
    if case["call"] == "lossless":
        return "exact"
    if case["call"] == "dataflow":  # one fused multiply-add and one rounding per value: whole numbers have to be the same
        return {"rel": 1e-6 if case["precision"] == "fp32" else 1e-4, "max": 1e-2, "differ": 0.0}
    if case["precision"] == "fp32":
        return {"rel": 5e-3, "max": 0.5}
    return {"rel": 3e-2 if case["precision"] == "bf16" or case["call"] == "predict" else 2.4e-2, "max": 0.9}


# ---- the same in 64 bits ---------------------------------------------------------------------------------------------

def _conv64(x, w, stride):
    """NHWC cross-correlation with "same" padding for an odd kernel, as one matrix product per tap."""
    k = w.shape[1]
    n, h, wd, _ = x.shape
    p, q = (h - 1) // stride + 1, (wd - 1) // stride + 1
    if k > 1:
        x = torch.nn.functional.pad(x, (0, 0, k // 2, k // 2, k // 2, k // 2))
    y = None
    for i in range(k):
        for j in range(k):
            part = x[:, i:i + (p - 1) * stride + 1:stride, j:j + (q - 1) * stride + 1:stride, :]
            t = part.reshape(-1, part.shape[-1]) @ w[:, i, j, :].t()
            y = t if y is None else y + t
    return y.reshape(n, p, q, -1)


def _forward64(case, params, x, stats=None, kept=None):
    """Logits.  stats None: batch statistics, appended to `kept` as (mean, unbiased variance) where that is a list."""
    layers = iter(_layers(case))
    at = [0]
    seen = iter(stats) if stats is not None else None

    def take(*shape):
        n = math.prod(shape)
        at[0] += n
        return params[at[0] - n:at[0]].view(*shape)

    def conv(v):
        _, _, cin, cout, k, s, _, _, bn = next(layers)
        z = _conv64(v, take(cout, k, k, cin), s)
        if not bn:
            return z + take(cout)
        gamma, beta = take(cout), take(cout)
        if seen is not None:
            mean, var = next(seen)
        else:
            flat = z.reshape(-1, cout)
            mean, var = flat.mean(0), flat.var(0, unbiased=False)
            if kept is not None:
                kept.append((mean, var * (flat.shape[0] / max(1, flat.shape[0] - 1))))
        return gamma * (z - mean) / torch.sqrt(var + 1e-5) + beta

    body, head = _parse(case)
    c = case["channels"]
    for letter, n, s in body:
        if letter == "p":
            h, w = x.shape[1] // 2 * 2, x.shape[2] // 2 * 2
            v = x[:, :h, :w, :]
            x = torch.maximum(torch.maximum(v[:, 0::2, 0::2], v[:, 0::2, 1::2]), torch.maximum(v[:, 1::2, 0::2], v[:, 1::2, 1::2]))
            continue
        if letter in "cr":
            x = torch.relu(conv(x))
        else:
            v = torch.relu(conv(x))
            if letter == "n":
                v = torch.relu(conv(v))
            v = conv(v)
            x = torch.relu(v + (conv(x) if c != n or s != 1 else x))
        c = n
    feat = x.mean((1, 2)) if head == "gap" else x.reshape(x.shape[0], -1)
    _, _, cin, cout, *_ = next(layers)
    return feat @ take(cout, cin).t() + take(cout)


def exact(case, seed):
    d = _inputs(case, seed)
    if case["call"] == "lossless":
        return None
    if case["call"] in ("dataflow", "encoded"):
        scale, shift = _normalisation(case)
        f = torch.float32  # the constants as the call takes them
        x = d["pixels"].double() * torch.tensor(scale, dtype=f, device="cuda").double() + torch.tensor(shift, dtype=f, device="cuda").double()
        if case["call"] == "dataflow":
            return {"words": None, "decoded": x.reshape(case["batch"], -1)}
        d["x"] = x
    if work(case)["flops"] > 5e13 or work(case)["bytes"] > 6e10:
        return None
    params = d["params"].double()
    if case["call"] == "predict":
        with torch.no_grad():
            kept = []
            _forward64(case, params, d["seen"].double(), kept=kept)
            return {"logits": _forward64(case, params, d["x"].double(), stats=kept)}
    params.requires_grad_(True)
    loss = torch.nn.functional.cross_entropy(_forward64(case, params, d["x"].double()), d["y"].long())
    loss.backward()
    return {"loss": float(loss.detach()), "grads": params.grad}
