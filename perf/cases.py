"""Measured cases: the training work that a user of the library has it do, through the Python binding.

Two kinds of program are measured.
  pipeline  `Pipeline.run_device`: several mini-batches through all K stages on one GPU, in the schedule's order, under
            one of the three policies: "inplace" (the method: every task reads its worker's live weights), "vsync"
            (forward passes on the weight version they are tagged with) and "1f1b" (the comparison system).
  stage     ONE stage's training step as a process that owns a single stage issues it: N micro-batch forward passes
            (each hands its result to the next worker), the backward pass over the mini-batch, the update.
Four kinds of network: multilayer perceptrons, VGG-style convolutional networks, bottleneck residual networks and
pre-LayerNorm transformers, in fp32 and in bf16 with fp32 masters.  The sizes of the listed cases are those of the
repository's benchmark configurations and tests, beside a few ragged ones of the same kinds.

A run under way: weights are those of an initialisation, the momentum buffers are full of the steps before (Gaussian,
eight times the spread of the array that they move), and the learning rate is that of late training, so that any number
of passes over the same mini-batches stays a run that converges.

What is compared: losses, stage results and the updated state (masters, bf16 working copy, momentum, which holds the
step's gradient).  The gradient itself and the gradient handed to the worker below are compared where layers are smooth.
Behind ReLU layers they are not reproducible: which side of zero an activation lies on hangs on roundings, and two correct
orders of summation give bf16 weight gradients 1 to 20 per cent apart (0.1 to 1 per cent in fp32).  The stage cases of
ReLU networks are therefore first workers, which hand no gradient down.
"""
import math

import numpy as np
import torch

import paper_2410_14312_amd as tmps
from paper_2410_14312_amd import binding
from workloads.configs import (Config, affine, avgpool, bottleneck, conv, embedding, layernorm, linear, maxpool,
                               softmax_ce, stage_shapes, transformer_block)
from workloads.synth import fan_in, param_shapes

LR, MOMENTUM = 1e-4, 0.9
DEVICE = "cuda:0"


# ------------------------------------------------------------------------------------------------ the cases
def _mlp(**kw):
    return dict({"net": "mlp", "classes": 10}, **kw)


def _vgg(**kw):
    return dict({"net": "vgg", "size": 32, "c": 64, "fc": 4096, "classes": 10}, **kw)


def _resnet(**kw):
    return dict({"net": "resnet", "size": 224, "c": 64, "groups": 4, "blocks": 0, "classes": 1000}, **kw)


def _gpt(**kw):
    return dict({"net": "gpt", "s": 512, "d": 768, "heads": 12, "ffn": 3072, "vocab": 32000}, **kw)


def listed():
    return [
        # the smallest thing anybody runs: a two-stage MLP in fp32, where launches and hand-overs between stages are all
        _mlp(name="mlp_f32_tiny", mode="inplace", dtype="f32", M=32, N=4, K=2, batches=2, din=64, width=128, depth=3),
        # the small bf16 benchmark configuration: four stages of one or two layers
        _mlp(name="mlp_bf16_pipeline", mode="inplace", dtype="bf16", M=256, N=4, K=4, batches=4, din=3072, width=1024, depth=5),
        # fp32 training at ragged widths and a ragged batch, one stage to a process
        _mlp(name="mlp_f32_ragged_stage", mode="stage", stage=0, dtype="f32", M=235, N=5, K=1, batches=1, din=784, width=1000, depth=4),
        # VGG-16 on 32 x 32 images: the paper's network, the convolutional benchmark configuration
        _vgg(name="vgg16_pipeline", mode="inplace", dtype="bf16", M=128, N=4, K=4, batches=2),
        # the same network with the paper's own policy for forward passes
        _vgg(name="vgg16_vsync", mode="vsync", dtype="bf16", M=128, N=4, K=4, batches=2),
        # ResNet-50 on 224 x 224 images: large maps, elementwise and normalisation work
        _resnet(name="resnet50_pipeline", mode="inplace", dtype="bf16", M=64, N=8, K=4, batches=2),
        # the stem and the first group of bottleneck blocks of that network on a worker of its own
        _resnet(name="resnet50_stage", mode="stage", stage=0, dtype="bf16", M=64, N=8, K=4, batches=1),
        # a two-block transformer at the size of a smoke run: many short kernels
        _gpt(name="transformer_tiny_f32", mode="inplace", dtype="f32", M=8, N=4, K=2, batches=2, layers=2, s=32, d=64, heads=2, ffn=128, vocab=96),
        # GPT-2 small, the benchmark's default workload and the largest case
        _gpt(name="gpt2_small_pipeline", mode="inplace", dtype="bf16", M=16, N=8, K=4, batches=2, layers=12),
        # three blocks of it on a worker of its own
        _gpt(name="gpt2_small_stage", mode="stage", stage=1, dtype="bf16", M=16, N=8, K=4, batches=1, layers=12),
        # the comparison system on it: a backward pass and an update for every micro-batch
        _gpt(name="gpt2_small_1f1b", mode="1f1b", dtype="bf16", M=16, N=8, K=4, batches=1, layers=12),
        # the last worker of a smaller transformer with a ragged sequence length and an odd vocabulary
        _gpt(name="transformer_ragged_stage", mode="stage", stage=1, dtype="bf16", M=12, N=4, K=2, batches=1, layers=4, s=333, d=512, heads=8, ffn=2048, vocab=5003),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_once(rng):
    c = {"mode": rng.choice(["inplace", "inplace", "stage", "stage", "vsync", "1f1b"]), "dtype": rng.choice(["bf16", "bf16", "f32"])}
    net = rng.choice(["mlp", "vgg", "resnet", "gpt"])
    K, N = rng.randint(1, 4), rng.randint(1, 8)
    if net == "mlp":
        c.update(_mlp(M=N * _log(rng, 4, 256), din=_log(rng, 64, 4096), width=_log(rng, 64, 4096), depth=rng.randint(K + 1, 8), classes=_log(rng, 10, 1000)))
    elif net == "vgg":
        c.update(_vgg(M=N * _log(rng, 2, 32), size=rng.randint(32, 64), c=8 * rng.randint(2, 8), fc=_log(rng, 128, 4096), classes=_log(rng, 10, 200)))
    elif net == "resnet":
        K = min(K, 3)
        c.update(_resnet(M=N * _log(rng, 1, 16), size=rng.randint(32, 224), c=8 * rng.randint(1, 8), groups=rng.randint(K, 4), blocks=rng.randint(1, 3), classes=_log(rng, 10, 1000)))
        K = min(K, c["groups"])
    else:
        heads, dh = rng.randint(1, 12), rng.choice([64, 64, 64, 32])
        c.update(_gpt(M=N * rng.randint(1, 4), layers=K * rng.randint(1, 3), s=_log(rng, 16, 512), d=heads * dh, heads=heads, ffn=4 * heads * dh, vocab=_log(rng, 64, 32000)))
    c.update(N=N, K=K, batches=1 if c["mode"] == "stage" else rng.randint(1, 2 if net == "vgg" else 4))
    if c["mode"] == "stage":
        c["stage"] = rng.randrange(K) if net == "gpt" else 0
    return c


def draw(rng):
    """Another case: any network, policy and type, sizes over the listed range; none costs more than the largest."""
    most = work(next(c for c in listed() if c["name"] == "gpt2_small_pipeline"))["flops"]
    while True:
        c = _draw_once(rng)
        # (fp32 contractions run on the vector units, some twenty times slower than bf16 ones on the matrix units)
        if work(c)["flops"] * (20 if c["dtype"] == "f32" else 1) <= 0.8 * most:
            return c


# ------------------------------------------------------------------------------------------------ the networks
def _split(layers, K):
    """Consecutive, nearly equal runs of layers."""
    return [layers[i * len(layers) // K:(i + 1) * len(layers) // K] for i in range(K)]


def _config(c):
    K = c["K"]
    vocab, in_shape = 0, None
    if c["net"] == "mlp":
        widths = [c["din"]] + [c["width"]] * (c["depth"] - 1) + [c["classes"]]
        layers = [[linear(a, b, i + 2 < len(widths))] for i, (a, b) in enumerate(zip(widths, widths[1:]))]
        # the narrow output layer goes with the layer before it
        layers[-2:] = [layers[-2] + layers[-1]]
        stages, in_shape, classes = [sum(g, []) for g in _split(layers, K)], (c["din"],), c["classes"]
    elif c["net"] == "vgg":
        h, cin, parts = c["size"], 3, []
        for mult, n in ((1, 2), (2, 2), (4, 3), (8, 3), (8, 3)):
            part = []
            for _ in range(n):
                part.append(conv(h, h, cin, c["c"] * mult))
                cin = c["c"] * mult
            parts.append(part + [maxpool(h, h, cin)])
            h //= 2
        parts = [parts[0] + parts[1], parts[2], parts[3],
                 parts[4] + [linear(h * h * cin, c["fc"], True), linear(c["fc"], c["fc"], True), linear(c["fc"], c["classes"], False)]]
        stages, in_shape, classes = [sum(g, []) for g in _split(parts, K)], (c["size"], c["size"], 3), c["classes"]
    elif c["net"] == "resnet":
        size, w = c["size"], c["c"]
        h = (size + 6 - 7) // 2 + 1
        stem = [conv(size, size, 3, w, 7, 2, 3, False), affine(h, h, w, True), maxpool(h, h, w, 3, 2, 1)]
        h = (h + 2 - 3) // 2 + 1
        cin, parts = w, []
        for g, nb in enumerate((3, 4, 6, 3)[:c["groups"]]):
            part = stem if g == 0 else []
            for b in range(c["blocks"] or nb):
                ls, h, cin = bottleneck(h, cin, w << g, 2 if (b == 0 and g > 0) else 1, b == 0)
                part = part + ls
            parts.append(part)
        parts[-1] = parts[-1] + [avgpool(h, h, cin), linear(cin, c["classes"], False)]
        stages, in_shape, classes = [sum(g, []) for g in _split(parts, K)], (size, size, 3), c["classes"]
    else:
        s, d, vocab = c["s"], c["d"], c["vocab"]
        blocks = [transformer_block(s, d, c["heads"], c["ffn"]) for _ in range(c["layers"])]
        stages = [sum(g, []) for g in _split(blocks, K)]
        stages[0] = [embedding(vocab, s, d)] + stages[0]
        stages[-1] = stages[-1] + [layernorm(d, s), linear(d, vocab, False, rows=s)]
        in_shape, classes = (s,), vocab
    rows = c["s"] if c["net"] == "gpt" else 1
    stages[-1] = stages[-1] + [softmax_ce(classes, rows=rows)]
    return Config(name=c["net"], dtype=c["dtype"], M=c["M"], N=c["N"], stages=stages, in_shape=in_shape, classes=classes, seed=0, lr=LR,
                  momentum=MOMENTUM, vocab=vocab)


def _flops(sp, first):
    """Floating point operations of one sample: forward, weight gradient and, unless nobody wants it, input gradient."""
    passes = 2 if first else 3
    if sp["kind"] == "linear":
        return passes * 2.0 * sp["rows"] * sp["din"] * sp["dout"]
    if sp["kind"] == "conv":
        ho = (sp["h"] + 2 * sp["pad"] - sp["r"]) // sp["stride"] + 1
        return passes * 2.0 * ho * ho * sp["cout"] * sp["r"] * sp["s"] * sp["cin"]
    if sp["kind"] == "attention":   # visible pairs: two products forward, five backward
        return 7 * sp["s"] * (sp["s"] + 1) * float(sp["d"])
    return 0.0


def work(case):
    cfg = _config(case)
    which = [case["stage"]] if case["mode"] == "stage" else range(cfg.K)
    samples = case["M"] * case["batches"]
    updates = case["batches"] * (case["N"] if case["mode"] == "1f1b" else 1)
    a = 2 if cfg.dtype == "bf16" else 4
    shapes = stage_shapes(cfg)
    flops = nbytes = 0.0
    for k in which:
        flops += samples * sum(_flops(sp, k == 0 and i == 0) for i, sp in enumerate(cfg.stages[k]))
        P = sum(int(np.prod(v)) for sp in cfg.stages[k] for v in param_shapes(sp).values())
        # an update reads and writes masters and momentum and writes the gradient (and the bf16 working copy)
        nbytes += updates * P * (20 + (2 if a == 2 else 0))
        if k == 0:
            nbytes += samples * np.prod(cfg.in_shape) * (4 if cfg.vocab else a)
        if case["mode"] == "stage":   # what comes from and goes to the neighbours, forward and backward
            n_in, n_out = int(np.prod(shapes[k][0])), int(np.prod(shapes[k][1]))
            nbytes += samples * (2 * n_in * a if k > 0 else 0)
            nbytes += samples * (n_out * 4 if k == cfg.K - 1 else 2 * n_out * a)
    return {"bytes": float(nbytes), "flops": float(flops)}


def tolerance(case):
    if case["dtype"] == "f32":   # sums of fp32 products; behind ReLU layers an activation next to zero moves whole gradients
        return {"gpt": {"rel": 2e-5, "max": 1e-3}, "mlp": {"rel": 2e-4, "max": 0.1}, "resnet": {"rel": 1e-3, "max": 0.3},
                "vgg": {"rel": 4e-3, "max": 0.5}}[case["net"]]
    # bf16 activations and gradients between layers, rounded on slightly different sums; a ReLU mask or a pooling winner
    # that such a difference decides moves single elements by their whole size
    return {"rel": 3e-2 if case["net"] == "vgg" else 2e-2, "max": 0.99}


# ------------------------------------------------------------------------------------------------ prepare and run
def _parameters(specs, gen):
    """Per-layer host arrays: He-normal weights, unit gains, N(0, 0.02^2) embedding tables, small biases and shifts."""
    out = []
    for sp in specs:
        p = {}
        for key, shape in param_shapes(sp).items():
            v = torch.randn(shape, generator=gen, device=DEVICE)
            if sp["kind"] == "embedding":
                v *= 0.02
            elif key == "w" and sp["kind"] in ("layernorm", "affine"):
                v = v.mul_(0.02).add_(sp.get("init_gain", 1.0))
            elif key == "w":
                v *= math.sqrt(2.0 / fan_in(sp))
            else:
                v *= 0.02
            p[key] = v.cpu().numpy()
        out.append(p)
    return out


def _region(st, index, first, count, dtype=torch.float32):
    """`count` values of a device region of the stage from value `first` on (the layouts that tmps_stage_bytes states)."""
    size = torch.empty(0, dtype=dtype).element_size()
    return st.regions[index][first * size:(first + count) * size].view(dtype)


def _past_steps(st, gen):
    """Momentum of the steps before: per array Gaussian, eight times the spread of the array's values."""
    mom = _region(st, 1, 0, st.P)
    for layer in range(len(st.specs)):
        for which in (0, 1):
            off, count = st.param_offset(layer, which)
            if count:
                spread = _region(st, 0, off, count).std(correction=0)
                mom[off:off + count] = torch.randn(count, generator=gen, device=DEVICE) * (8.0 * spread)


def _state_of(st):
    """What a stage's pass leaves behind: master parameters, bf16 working copy, momentum and, on smooth layers, gradient."""
    out = {"masters": _region(st, 0, 0, st.P), "momentum": _region(st, 1, 0, st.P)}
    if all(sp["kind"] != "embedding" and not sp.get("relu") for sp in st.specs):
        out["gradient"] = _region(st, 1, st.P, st.P)
    if st.cfg.dtype == binding.TMPS_BF16_F32MASTER:
        out["working_copy"] = _region(st, 0, 2 * st.P, st.P, torch.bfloat16)
    return out


def prepare(case, seed):
    cfg = _config(case)
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(int(seed))
    host = np.random.default_rng(int(seed))
    M, N, n = case["M"], case["N"], case["batches"]
    rows = case["s"] if case["net"] == "gpt" else 1
    if cfg.vocab:
        tokens = host.integers(0, cfg.vocab, size=(n * M, rows + 1), dtype=np.int32)
        x, labels = np.ascontiguousarray(tokens[:, :-1]), np.ascontiguousarray(tokens[:, 1:])
    else:
        x = torch.randn((n * M,) + tuple(cfg.in_shape), generator=gen, device=DEVICE).cpu().numpy()
        labels = host.integers(0, cfg.classes, size=(n * M,), dtype=np.int32)
    s = {"case": case, "mode": case["mode"]}
    if case["mode"] == "stage":
        k = case["stage"]
        st = tmps.Stage(cfg.stages[k], cfg.dtype, M // N, N, N, cfg.lr, cfg.momentum, borrow_input=True, device=DEVICE)
        st.set_params(_parameters(cfg.stages[k], gen))
        _past_steps(st, gen)
        act = dict(dtype=st.act_dtype, device=DEVICE)
        if k == 0:
            s["x"] = st.prepare_input(x).reshape(M, -1).contiguous()
        else:
            s["x"] = torch.randn(M, st.in_elems, generator=gen, device=DEVICE).to(st.act_dtype)
            s["dx"] = torch.empty(M, st.in_elems, **act)
        if st.is_last:
            s["labels"] = torch.from_numpy(labels).to(DEVICE).reshape(M, -1)
            s["losses"] = torch.zeros(N, device=DEVICE)
            s["y"] = torch.empty(M, st.out_elems, device=DEVICE)
        else:
            s["dy"] = (torch.randn(M, st.out_elems, generator=gen, device=DEVICE) / (M * math.sqrt(st.out_elems))).to(st.act_dtype)
            s["y"] = torch.empty(M, st.out_elems, **act)
        s["stage"] = st
    else:
        params = [_parameters(specs, gen) for specs in cfg.stages]
        pipe = tmps.Pipeline(cfg, params, device=DEVICE, vertical_sync=case["mode"] == "vsync", baseline_1f1b=case["mode"] == "1f1b")
        for st in pipe.stages:
            _past_steps(st, gen)
        s["x"], s["labels"] = pipe.upload([(x, labels)])
        s["runs"] = n * (N if case["mode"] == "1f1b" else 1)
        s["losses"] = torch.zeros(s["runs"], device=DEVICE)
        s["pipe"] = pipe
    return s


def run(state):
    s = state
    if s["mode"] != "stage":
        s["pipe"].run_device(s["x"], s["labels"], s["runs"], s["losses"], want_log=False)
        return {"losses": s["losses"], "stages": [_state_of(st) for st in s["pipe"].stages]}
    st = s["stage"]
    mb, N = st.micro, st.N
    for j in range(N):
        rows = slice(j * mb, (j + 1) * mb)
        if st.is_last:
            st.forward_micro(j, s["x"][rows], y=s["y"][rows], labels=s["labels"][rows], loss_out=s["losses"][j:j + 1])
        else:
            st.forward_micro(j, s["x"][rows], y=s["y"][rows])
    st.backward(list(range(N)), dy=s.get("dy"), dx=s.get("dx"))
    st.update()
    return dict(_state_of(st), y=s["y"], dx=s.get("dx"), losses=s.get("losses"))
