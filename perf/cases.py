"""Timing cases of the library: what a training job built on it does, pass by pass.

Three kinds of pass:
  step     one worker's training step: spb_forward to the loss, then spb_backward_truncated over the top `depth` units.
           Perceptrons, residual CNNs and Transformer encoders; launched call by call ("eager"), replayed from a HIP
           graph the program captured once ("graph"), or on the library's own workspace ("static").
  update   the server's side of an iteration: spb_aggregate_update over the partial gradients of several workers.
  place    the scheduler's side: spb_schedule_tasks over a mix of jobs (host data in, host data out).

A worker's gradients lie in one float32 buffer, as a program that sends them keeps them; a step's result is its loss and
the stretch of that buffer each visited unit fills.
"""
from __future__ import annotations

import math
import random

import torch

import paper_2111_10672_amd as spb


def listed():
    return [
        # The smallest step: a float32 perceptron (784-256-256-256-10, batch 64), half of it backpropagated, launched call
        # by call on the library's own workspace.  Launch latency is all of it.
        dict(name="mlp_f32_static", task="step", family="mlp", dtype="f32", batch=64, dims="784,256,256,256,10", depth=2, launch="static"),
        # Eight layers of 1024 at batch 256, the last worker's complete pass, replayed from a HIP graph.
        dict(name="mlp_1024_graph", task="step", family="mlp", dtype="bf16", batch=256, dims="1024,1024,1024,1024,1024,1024,1024,1024,100", depth=8,
             launch="graph"),
        # Widths and a batch that are whole tiles of nothing, several thousand classes.
        dict(name="mlp_ragged", task="step", family="mlp", dtype="bf16", batch=1000, dims="1336,2008,1000,504,4999", depth=3, launch="eager"),
        # A perceptron with the matrix shapes of a Transformer layer.
        dict(name="mlp_wide", task="step", family="mlp", dtype="bf16", batch=4096, dims="768,3072,2304,768,24", depth=4, launch="eager"),
        # ResNet-18-style on 32x32 images: all but the stem backpropagated.
        dict(name="resnet18_32px", task="step", family="resnet_basic", batch=128, image=32, stem="3x3", blocks="2,2,2,2", widths="64,128,256,512",
             classes=10, depth=9),
        # ResNet-50-style on 224x224 images: all but the stem backpropagated.
        dict(name="resnet50_224px", task="step", family="resnet_bottleneck", batch=64, image=224, stem="7x7", blocks="3,4,6,3",
             widths="256,512,1024,2048", classes=1000, depth=17),
        # The 35-unit bottleneck stack on 32x32 images, an early worker's short backward pass: mostly the forward direction.
        dict(name="resnet101_32px_shallow", task="step", family="resnet_bottleneck", batch=64, image=32, stem="3x3", blocks="3,4,23,3",
             widths="256,512,1024,2048", classes=10, depth=4),
        # BERT-base shapes, 32 sequences of 128, everything but the embedding backpropagated.
        dict(name="encoder_128", task="step", family="encoder", batch=32, seq=128, layers=12, hidden=768, ffn=3072, vocab=30522, loss_rows=614, depth=13),
        # The same model at its longest sequences.
        dict(name="encoder_512", task="step", family="encoder", batch=8, seq=512, layers=12, hidden=768, ffn=3072, vocab=30522, loss_rows=614, depth=13),
        # A small batch of odd length, half of the layers: few rows under every product.
        dict(name="encoder_ragged", task="step", family="encoder", batch=7, seq=72, layers=12, hidden=768, ffn=3072, vocab=30522, loss_rows=75, depth=7),
        # The server's update of the encoder from four workers at depths ceil(j L / 4).
        dict(name="update_encoder", task="update", family="encoder", batch=32, seq=128, layers=12, hidden=768, ffn=3072, vocab=30522, loss_rows=614,
             workers=4),
        # A scheduling interval: 200 jobs on 45 devices.
        dict(name="place_200_jobs", task="place", jobs=200, machines=45, longest=120, gang=False),
    ]


def draw(rng: random.Random):
    limit = max(work(c)["flops"] for c in listed())
    task = rng.choice(["step"] * 7 + ["update", "place"])
    if task == "place":
        # (gangs on a wide cluster take longer per task: fewer of them)
        gang = rng.random() < 0.25
        return dict(task="place", jobs=_log(rng, 10, 60 if gang else 180), machines=rng.randint(16, 48), longest=rng.randint(20, 60 if gang else 120), gang=gang)
    while True:
        family = rng.choice(["mlp", "mlp", "resnet", "encoder", "encoder"])
        case = {"mlp": _draw_mlp, "resnet": _draw_resnet, "encoder": _draw_encoder}[family](rng)
        if task == "update":
            case = {k: v for k, v in case.items() if k not in ("depth", "launch")}
            case.update(task="update", workers=rng.randint(1, 8))
            if sum(n for _, n in _shape(case)[1]) <= 1.3e8:
                return case
            continue
        case["task"] = "step"
        if work(case)["flops"] <= limit:
            return case


def _log(rng, lo, hi, step=1):
    """An integer in [lo, hi], uniform over the logarithm, a multiple of `step`."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / step)) * step))


def _draw_mlp(rng):
    f32 = rng.random() < 0.3
    layers = rng.randint(2, 10)
    hi = 1024 if f32 else 4096
    step = 4 if f32 else 8          # widths are whole 16-byte chunks
    if rng.random() < 0.5:
        dims = [_log(rng, 64, hi, step)] * layers
    else:
        dims = [_log(rng, 64, hi, step) for _ in range(layers)]
    batch = _log(rng, 32, 1024 if f32 else 8192)
    classes = _log(rng, 2, 5000)
    case = dict(family="mlp", dtype="f32" if f32 else "bf16", batch=batch, dims=",".join(map(str, dims + [classes])), depth=rng.randint(1, layers))
    # what fits the library's own workspace may run there
    fits = (layers + 5) * (batch * (max(dims) + 8) * (4 if f32 else 2) + 256) + 8 * batch * (classes + 8) <= spb.SPB_STATIC_WORKSPACE_BYTES
    case["launch"] = rng.choice(["eager", "graph", "static"] if fits else ["eager", "graph"])
    return case


def _draw_resnet(rng):
    bottleneck = rng.random() < 0.5
    blocks = rng.choice(["1,1,1,1", "2,2,2,2", "3,4,6,3", "3,4,23,3"] if bottleneck else ["1,1,1,1", "2,2,2,2", "3,4,6,3"])
    base = rng.choice([32, 48, 64]) * (4 if bottleneck else 1)
    small = rng.random() < 0.5      # 3x3 stem on small images, or 7x7 stem with pooling on large ones
    image = rng.randint(16, 64) if small else rng.randint(96, 255)
    n_units = 2 + sum(map(int, blocks.split(",")))
    # depths as the configurations' sweeps have them: the stem stays below the cut
    return dict(family="resnet_bottleneck" if bottleneck else "resnet_basic", batch=_log(rng, 4, 256), image=image, stem="3x3" if small else "7x7",
                blocks=blocks, widths=",".join(str(base << i) for i in range(4)), classes=_log(rng, 5, 1000), depth=rng.randint(1, n_units - 1))


def _draw_encoder(rng):
    seq = _log(rng, 16, 512, 8)
    batch = _log(rng, 1, max(1, min(64, 8192 // seq)))
    layers = rng.randint(1, 12)
    hidden = 64 * rng.randint(2, 16)
    return dict(family="encoder", batch=batch, seq=seq, layers=layers, hidden=hidden, ffn=hidden * rng.choice([2, 3, 4]), vocab=_log(rng, 1000, 30522),
                loss_rows=max(1, batch * seq * 15 // 100), depth=rng.randint(1, layers + 2))


# ---- model shapes --------------------------------------------------------------------------------------------------

def _config(case):
    """The library's model description of a step or update case."""
    family = case["family"]
    if family == "mlp":
        return dict(family="mlp", dtype=case["dtype"], batch=case["batch"], dims=[int(d) for d in case["dims"].split(",")])
    if family.startswith("resnet"):
        widths = [int(w) for w in case["widths"].split(",")]
        stem_width = widths[0] // 4 if family == "resnet_bottleneck" else widths[0]
        stem = dict(kernel=3, stride=1, pad=1, pool=False) if case["stem"] == "3x3" else dict(kernel=7, stride=2, pad=3, pool=True)
        return dict(family=family, dtype="bf16", batch=case["batch"], image=[case["image"], case["image"], 3], stem=dict(stem, width=stem_width),
                    stage_blocks=[int(b) for b in case["blocks"].split(",")], stage_widths=widths, classes=case["classes"])
    return dict(family="encoder", dtype="bf16", heads=case["hidden"] // 64,
                **{k: case[k] for k in ("batch", "seq", "layers", "hidden", "ffn", "vocab", "loss_rows")})


def _shape(case):
    """(units, [(unit, elements) of each parameter], products, input elements) of a case's model; a product is
    (unit, rows, columns, reduction, forms an input gradient when its unit does, has a weight gradient)."""
    cfg, params, prods = _config(case), [], []
    if cfg["family"] == "mlp":
        dims = cfg["dims"]
        for u, (i, o) in enumerate(zip(dims, dims[1:])):
            params += [(u, i * o), (u, o)]
            prods.append((u, cfg["batch"], o, i, u > 0, True))
        return len(dims) - 1, params, prods, cfg["batch"] * dims[0]
    if cfg["family"] == "encoder":
        rows, h, f, seq = cfg["batch"] * cfg["seq"], cfg["hidden"], cfg["ffn"], cfg["seq"]
        params += [(0, cfg["vocab"] * h), (0, seq * h)]
        for u in range(1, cfg["layers"] + 1):
            for i, o in ((h, 3 * h), (h, h), (h, f), (f, h)):
                params += [(u, i * o), (u, o)]
                prods.append((u, rows, o, i, True, True))
            params += [(u, h)] * 4
            prods += [(u, rows, seq, h, True, True), (u, rows, h, seq, True, True)]     # scores and context: both operands get gradients
        u = cfg["layers"] + 1
        params += [(u, h), (u, h), (u, cfg["vocab"] * h), (u, cfg["vocab"])]
        prods.append((u, cfg["loss_rows"], cfg["vocab"], h, True, True))
        return u + 1, params, prods, rows
    st, n, hw = cfg["stem"], cfg["batch"], cfg["image"][0]
    unit_in = n * hw * hw * 3

    def conv(unit, size, cin, cout, k, stride, pad, dx=True):
        out = (size + 2 * pad - k) // stride + 1
        params.extend([(unit, cout * k * k * cin), (unit, cout), (unit, cout)])
        prods.append((unit, n * out * out, cout, k * k * cin, dx, True))
        return out

    hw = conv(0, hw, 3, st["width"], st["kernel"], st["stride"], st["pad"], dx=False)
    hw = (hw - 1) // 2 + 1 if st["pool"] else hw
    unit, cin = 0, st["width"]
    for stage, (count, width) in enumerate(zip(cfg["stage_blocks"], cfg["stage_widths"])):
        for j in range(count):
            unit += 1
            stride = 2 if stage > 0 and j == 0 else 1
            if stride != 1 or cin != width:
                conv(unit, hw, cin, width, 1, stride, 0)
            if cfg["family"] == "resnet_bottleneck":
                conv(unit, hw, cin, width // 4, 1, 1, 0)
                hw = conv(unit, hw, width // 4, width // 4, 3, stride, 1)
                conv(unit, hw, width // 4, width, 1, 1, 0)
            else:
                hw = conv(unit, hw, cin, width, 3, stride, 1)
                conv(unit, hw, width, width, 3, 1, 1)
            cin = width
    params += [(unit + 1, cfg["classes"] * cin), (unit + 1, cfg["classes"])]
    prods.append((unit + 1, n, cfg["classes"], cin, True, True))
    return unit + 2, params, prods, unit_in


def _depths(case):
    """An update case's workers: worker j of n backpropagated ceil(j L / n) units."""
    n_units = _shape(case)[0]
    return [-(-j * n_units // case["workers"]) for j in range(1, case["workers"] + 1)]


def work(case):
    if case["task"] == "place":
        tasks = sum(len(j["durations"]) * j["iterations"] for j in _jobs(case, 0))
        return {"bytes": 48 * tasks, "flops": 0}       # one record per task
    n_units, params, prods, n_in = _shape(case)
    size = 4 if case.get("dtype") == "f32" else 2
    if case["task"] == "update":
        nbytes = flops = 0
        depths = _depths(case)
        for unit, numel in params:
            c = sum(1 for k in depths if unit >= n_units - k)
            if c:
                nbytes += numel * (4 * c + 8 + 2 * size)
                flops += numel * (c + 6)
        return {"bytes": nbytes, "flops": flops}
    cut = n_units - case["depth"]
    flops = nbytes = 0
    for unit, m, n, k, dx, dw in prods:
        # the lowest visited unit of a perceptron hands no gradient down; inside a wider unit only its first product does not
        inner = dx and (unit > cut or (unit == cut and case["family"] != "mlp" and unit != n_units - 1))
        flops += 2 * m * n * k * (1 + (1 if unit >= cut and dw else 0) + (1 if inner else 0))
    for unit, numel in params:
        nbytes += numel * size + (4 * numel if unit >= cut else 0)
    nbytes += n_in * (4 if case["family"] == "encoder" else size) + 4
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    if case["task"] == "place":
        return "exact"
    if case["task"] == "update":
        # float32 sums; a bfloat16 parameter may land on the other side of a rounding boundary (one step, 2^-8)
        return {"rel": 1e-4, "max": 1e-2}
    if case.get("dtype") == "f32":
        return {"rel": 1e-5, "max": 1e-3}
    if case["family"] == "encoder":
        return {"rel": 1e-2, "max": 0.4}
    # bfloat16 storage between ReLU layers: a pre-activation that two correct implementations round to different sides
    # of zero switches a whole term of a gradient sum on or off, and such flips add up from layer to layer (the exact
    # and the storage-rounded float64 oracle are 2 to 8 % apart on the lowest layers of the deep configurations)
    return {"rel": 3e-2, "max": 0.9}


# ---- inputs --------------------------------------------------------------------------------------------------------

def _jobs(case, seed):
    """Jobs as a profile of the library would describe them: a complete step of 0.1 to 6 ms of which a third is the
    forward pass, worker j of W at depth ceil(j / W), worker counts in the proportions 50 / 10 / 20 / 15 / 5 % of
    1 / 2 / 4 / 8 / 16.  Iteration and worker counts come from the case alone, times and sizes from the seed."""
    fixed = random.Random(f"{case['jobs']} {case['machines']} {case['longest']} {case['gang']}")
    rng = random.Random(seed)
    jobs = []
    for _ in range(case["jobs"]):
        u = fixed.random()
        w = 1 if u < 0.5 else 2 if u < 0.6 else 4 if u < 0.8 else 8 if u < 0.95 else 16
        iters = fixed.randint(max(1, case["longest"] // 6), case["longest"])
        full, mem = 10 ** rng.uniform(-4.0, -2.2), 10 ** rng.uniform(-3.5, -1.5)
        jobs.append(dict(arrival=rng.uniform(0.0, 2.0), iterations=iters, model_size=10 ** rng.uniform(6.0, 8.5),
                         durations=[full * (1 + 2 * j / w) / 3 for j in range(1, w + 1)],
                         resources=[mem * (0.4 + 0.6 * j / w) for j in range(1, w + 1)]))
    return jobs


def _slab(counts, dtype, device):
    """One zeroed buffer with room for every count (each on a 256-byte boundary) and the offset of each."""
    step = 256 // torch.empty((), dtype=dtype).element_size()
    offsets, end = [], 0
    for c in counts:
        offsets.append(end)
        end += -(-c // step) * step
    return torch.zeros(end, dtype=dtype, device=device), offsets


class _State:
    pass


def prepare(case, seed):
    s = _State()
    s.case = case
    if case["task"] == "place":
        s.jobs = _jobs(case, seed)
        return s
    device = torch.device("cuda:0")
    gen = torch.Generator(device=device).manual_seed(seed)
    cfg = _config(case)
    dtype = torch.float32 if cfg["dtype"] == "f32" else torch.bfloat16

    def normal(shape, std, mean=0.0):
        return torch.randn(shape, generator=gen, device=device) * std + mean

    # parameters, all in one buffer: fan-in scaled weights (0.02 in an encoder), biases and shifts around 0, scales
    # around 1 - around 1/4 on the affine that closes a residual branch, as training leaves it
    handle = spb.spb_model_create(spb.desc_from_config(cfg))
    infos = [spb.spb_param_info(handle, i) for i in range(spb.spb_param_count(handle))]
    spb.spb_model_destroy(handle)
    numels = [i["numel"] for i in infos]
    s.params, at = _slab(numels, dtype, device)
    closing = "aff3.scale" if cfg["family"] == "resnet_bottleneck" else "aff2.scale"
    params = {}
    for info, off in zip(infos, at):
        name, shape = info["name"], info["shape"]
        if len(shape) > 1:
            fan_in = info["numel"] // shape[0]
            value = normal(shape, 0.02 if cfg["family"] == "encoder" else math.sqrt(2.0 / fan_in))
        elif name.endswith(".scale") or (".ln" in name and name.endswith(".weight")):
            mean = 0.25 if name.endswith(closing) else 1.0
            value = normal(shape, 0.1 * mean, mean)
        else:
            value = normal(shape, 0.02)
        view = s.params[off:off + info["numel"]].view(shape)
        view.copy_(value)
        params[name] = view
    s.model = model = spb.SpbModel(cfg, params, device)

    if case["task"] == "update":
        s.depths = _depths(case)
        s.velocity, at = _slab(numels, torch.float32, device)
        s.velocity.copy_(normal(s.velocity.shape, 0.01))
        s.velocities = [s.velocity[o:o + n].view(i["shape"]) for o, n, i in zip(at, numels, infos)]
        s.grads = []
        for _ in s.depths:
            slab = normal(s.velocity.shape, 0.01)
            s.grads.append([slab[o:o + n].view(i["shape"]) for o, n, i in zip(at, numels, infos)])
        return s

    s.grad_slab, at = _slab(numels, torch.float32, device)
    model.grads = [s.grad_slab[o:o + n].view(i["shape"]) for o, n, i in zip(at, numels, infos)]
    spb.spb_bind_grads(model.handle, model.grads)
    bounds = at + [s.grad_slab.numel()]
    first = [next(j for j, i in enumerate(infos) if i["unit"] == u) for u in range(model.n_units)] + [len(infos)]
    s.result = [model.loss] + [s.grad_slab[bounds[first[u]]:bounds[first[u + 1]]] for u in range(model.n_units - case["depth"], model.n_units)]

    def integers(hi, n):
        return torch.randint(0, hi, (n,), generator=gen, device=device, dtype=torch.int32)

    if cfg["family"] == "encoder":
        tokens = cfg["batch"] * cfg["seq"]
        s.batch = {"x": integers(cfg["vocab"], tokens).view(cfg["batch"], cfg["seq"]), "labels": integers(cfg["vocab"], cfg["loss_rows"]),
                   "loss_rows": torch.randperm(tokens, generator=gen, device=device)[:cfg["loss_rows"]].to(torch.int32)}
    else:
        shape = (cfg["batch"], cfg["dims"][0]) if cfg["family"] == "mlp" else (cfg["batch"], *cfg["image"])
        classes = cfg["dims"][-1] if cfg["family"] == "mlp" else cfg["classes"]
        s.batch = {"x": normal(shape, 1.0).to(dtype), "labels": integers(classes, cfg["batch"])}
    launch, k = case.get("launch", "eager"), case["depth"]
    if launch != "static":
        model.reserve(k)
    if launch == "graph":
        stream = torch.cuda.Stream()
        stream.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(stream):
            model.step(s.batch, k)
            stream.synchronize()
            s.graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(s.graph, stream=stream):
                model.step(s.batch, k)
    return s


def run(s):
    case = s.case
    if case["task"] == "place":
        placed, makespan = spb.spb_schedule_tasks(s.jobs, case["machines"], gamma=1.0 / 50e9, gang=case["gang"])
        return {"makespan": makespan, "machine": torch.tensor([t["machine"] for t in placed], dtype=torch.int32),
                "start": torch.tensor([t["start"] for t in placed], dtype=torch.float64)}
    model = s.model
    if case["task"] == "update":
        spb.spb_aggregate_update(model.handle, s.depths, s.grads, s.velocities, 0.01, 0.9, 1e-4, True, model.stream())
        return [s.params, s.velocity]
    launch, k = case.get("launch", "eager"), case["depth"]
    if launch == "graph":
        s.graph.replay()
    elif launch == "static":
        model.forward_static(s.batch, k)
        model.backward(k)
    else:
        model.step(s.batch, k)
    return s.result
