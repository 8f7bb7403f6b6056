"""The work that users of this framework have it do, as cases to time and to compare.

A case is one pass of a training or validation program on one GPU: a training step (forward, loss,
backward, update) of a convolutional network or of a Vision Transformer, or the forward pass of a
validation batch.  The networks are the ones of `workloads` (the sizes of the benchmark and of the
configurations); batch sizes run from a single image to the benchmark's.  A pass goes through
`StepRunner`, `Trainer`, `VitRunner` and the two evaluation entry points, as the epoch loop calls them.

Values: images N(0, 1), labels uniform, convolution weights He-normal, everything else near its usual
starting value; the batch norm that ends a residual branch has a gain of 0.2, the momentum buffers hold
what earlier steps leave there, and validation runs on running statistics that fit the network.
Parameters of one kind lie in one flat buffer, as in a program that exchanges or saves them in large
pieces, and are returned whole.  A convolutional step returns its gradients as part of the momentum
buffers: at bf16 storage two correct implementations differ by up to 28 % in the weight gradients of the
deepest network (ReLU decisions on values that differ by a rounding, amplified by the batch norms).
"""
import math

import torch

import workloads as WL
from paper_2503_23186_amd import cnnk
from paper_2503_23186_amd.runner import StepRunner
from paper_2503_23186_amd.trainer import Trainer
from paper_2503_23186_amd.vit import VitRunner, cnnk_vit_eval_step

DEVICE = "cuda:0"
CNN_LR, VIT_LR, MOMENTUM, WEIGHT_DECAY = 3e-3, 1e-3, 0.9, 5e-4
# rms of the momentum buffers at batch 128 (it goes with 1/sqrt(batch), as the gradients' noise does)
MOM = {"conv_w": 4e-2, "fc_w": 1e-1, "bn_gamma": 1e-1, "bn_beta": 1e-1, "fc_b": 1e-1}
DATASET = 4096                # images that the epoch loop's case draws its mini-batches from

CNNS = {"tiny": WL.tiny_cnn, "vgg": WL.vgg_style, "resnet18": WL.resnet18, "resnet50": WL.resnet50, "wrn": WL.wrn28_10}


def _cnn(name, net, batch, dtype="bf16", mode="train"):
    return {"name": name, "kind": "cnn", "net": net, "batch": batch, "dtype": dtype, "mode": mode}


def _vit(name, batch, image, patch, dim, layers, dtype="bf16", mode="train"):
    return {"name": name, "kind": "vit", "batch": batch, "image": image, "patch": patch, "dim": dim, "layers": layers,
            "dtype": dtype, "mode": mode}


def listed():
    return [
        # the smallest program: three layers in fp32, all latency
        _cnn("tiny_f32_b8", "tiny", 8, "f32"),
        # the epoch loop's mini-batch: gather out of a resident data set, then the step of a plain network
        _cnn("vgg_epoch_b128", "vgg", 128, mode="epoch"),
        # the benchmark
        _cnn("resnet18_b256", "resnet18", 256),
        # one replica's share of that batch on eight devices
        _cnn("resnet18_b32", "resnet18", 32),
        # the ragged last batch of an epoch (50 000 images in batches of 193 leave 13; 77 is odd in every tile)
        _cnn("resnet18_b77", "resnet18", 77),
        # deep, wide-tensor networks at their configurations' sizes: bandwidth-bound, and the largest convolutions
        _cnn("resnet50_b256", "resnet50", 256),
        _cnn("wrn_b128", "wrn", 128),
        # validation: 10 000 images in batches of 200
        _cnn("resnet50_eval_b200", "resnet50", 200, mode="eval"),
        # the second model family at its configuration's size
        _vit("vit_b16_b64", 64, 224, 16, 768, 12),
        # one replica's share of it, and a request of a few images
        _vit("vit_b16_b8", 8, 224, 16, 768, 12),
        _vit("vit_b16_eval_b4", 4, 224, 16, 768, 12, mode="eval"),
        # a transformer of half the width on images at their own size: 65 tokens
        _vit("vit_small_b96", 96, 32, 4, 384, 6),
    ]


def _log(rng, low, high):
    return max(low, min(high, round(math.exp(rng.uniform(math.log(low), math.log(high))))))


def draw(rng):
    kind = rng.choice(("tiny", "vgg", "resnet18", "resnet18", "resnet50", "wrn", "vit_b16", "vit_small"))
    mode = rng.choice(("train", "train", "eval"))
    if kind == "tiny":
        c = _cnn("", kind, _log(rng, 1, 512), "f32", mode)
    elif kind == "vgg":
        c = _cnn("", kind, _log(rng, 16, 512), "bf16", rng.choice(("train", "epoch", "eval")))
    elif kind in CNNS:
        c = _cnn("", kind, _log(rng, 16, {"resnet18": 512, "resnet50": 256, "wrn": 128}[kind]), "bf16", mode)
    elif kind == "vit_b16":
        c = _vit("", _log(rng, 1, 64), 224, 16, 768, 12, "bf16", mode)
    else:
        image, patch = rng.choice(((32, 4), (32, 8), (64, 8), (96, 8), (160, 16), (224, 16)))
        c = _vit("", _log(rng, 1, 192), image, patch, 64 * rng.randint(2, 8), rng.randint(2, 8), "bf16", mode)
    del c["name"]
    return c


# ---- networks ----------------------------------------------------------------------------------------
def _net(case):
    if case["kind"] == "cnn":
        return CNNS[case["net"]](batch=case["batch"], dtype=case["dtype"])
    d = case["dim"]
    return WL.ViT("vit", case["batch"], case["dtype"], case["image"], case["patch"], d, d // 64, case["layers"], 4 * d)


def _flat(kinds, tensors, pointers):
    """Move `tensors` (a runner's float buffers) into one flat buffer for each kind; the runner's list and
    pointers follow.  Kind None: there is no tensor.  Returns {kind: buffer}."""
    flat = {}
    for kind in dict.fromkeys(k for k in kinds if k is not None):
        mine = [k for k, name in enumerate(kinds) if name == kind]
        at = [0]
        for k in mine:
            at.append(at[-1] + (tensors[k].numel() + 63) // 64 * 64)
        flat[kind] = torch.zeros(at[-1], dtype=torch.float32, device=DEVICE)
        for k, first in zip(mine, at):
            tensors[k] = flat[kind][first:first + tensors[k].numel()].view(tensors[k].shape)
            pointers[k] = tensors[k].data_ptr()
    return flat


def _normal(t, gen, std=1.0, mean=0.0):
    t.copy_(torch.randn(t.shape, generator=gen, device=DEVICE).mul_(std).add_(mean))


def _cnn_values(net, run, gen):
    """Parameters, momentum and, from the expected second moment of every tensor, running statistics."""
    ends = {L["gamma"] for L in net.layers if L["op"] == "bn" and L["res"] >= 0}
    into_add = {L["a"] for L in net.layers if L["op"] == "add"}
    ends |= {L["w"] for L in net.layers if L["op"] == "conv" and L["y"] in into_add}
    for k, p in enumerate(net.params):
        kind, quiet = p["kind"], 0.2 if k in ends else 1.0
        if kind == "conv_w":
            _normal(run.param[k], gen, quiet * math.sqrt(2.0 / p["fan_in"]))
        elif kind == "fc_w":
            _normal(run.param[k], gen, math.sqrt(1.0 / p["fan_in"]))
        else:
            _normal(run.param[k], gen, 0.05 * quiet, quiet if kind == "bn_gamma" else 0.0)
        _normal(run.mom[k], gen, MOM[kind] * math.sqrt(128.0 / net.batch))
    moment = {0: 1.0}
    for i, L in enumerate(net.layers):
        if L["op"] == "conv":
            moment[L["y"]] = 2.0 * moment[L["x"]] * (0.04 if L["w"] in ends else 1.0)
        elif L["op"] == "bn":
            run.bn_running[i][0].copy_(torch.randn(L["C"], generator=gen, device=DEVICE).mul_(0.1 * math.sqrt(moment[L["x"]])))
            run.bn_running[i][1].copy_(torch.rand(L["C"], generator=gen, device=DEVICE).add_(0.5).mul_(moment[L["x"]]))
            out = (0.04 if L["gamma"] in ends else 1.0) + (moment[L["res"]] if L["res"] >= 0 else 0.0)
            moment[L["y"]] = out * (1.0 if L["res"] >= 0 or not L["relu"] else 0.5)
        elif L["op"] == "add":
            moment[L["y"]] = moment[L["a"]] + moment[L["b"]]
        elif L["op"] == "pool":
            moment[L["y"]] = moment[L["x"]]
    run.refresh_low_precision()


def _prepare_cnn(case, gen):
    net = _net(case)
    if case["mode"] == "epoch":
        trainer = Trainer(net, device=DEVICE)
        run = trainer.run
    else:
        trainer = None
        run = StepRunner(net.layers, net.slots, [p["shape"] for p in net.params], net.dtype, device=DEVICE)
    kinds = [p["kind"] for p in net.params]
    bns = ["running" if t is not None else None for t in run.bn_running]
    state = {"case": case, "run": run, "trainer": trainer, "param": _flat(kinds, run.param, run.buffers.param),
             "mom": _flat(kinds, run.mom, run.buffers.mom), "running": _flat(bns, run.bn_running, run.buffers.bn_running)}
    _cnn_values(net, run, gen)
    if trainer is not None:
        n, h, w, c = net.slots[0]
        state["x"] = torch.randn((DATASET, h, w, c), generator=gen, device=DEVICE).to(run.tdt)
        state["y"] = torch.randint(0, net.classes, (DATASET,), generator=gen, device=DEVICE).to(torch.int32)
        state["idx"] = torch.randperm(DATASET, generator=gen, device=DEVICE)[:n].contiguous()
    else:
        run.act[0].copy_(torch.randn(run.act[0].shape, generator=gen, device=DEVICE))
        run.labels.copy_(torch.randint(0, net.classes, run.labels.shape, generator=gen, device=DEVICE))
    if case["mode"] == "eval":
        state["correct"] = torch.zeros(1, dtype=torch.int32, device=DEVICE)
    return state


def _prepare_vit(case, gen):
    net = _net(case)
    run = VitRunner(net, device=DEVICE)
    kinds = [name.split(".")[0] for name in run.names]
    state = {"case": case, "run": run, "param": _flat(kinds, run.param, run.buffers.param),
             "grad": _flat(kinds, run.grad, run.buffers.grad)}
    for k, base in enumerate(kinds):
        _normal(run.param[k], gen, 0.1 if base[0] in "gb" and base != "be" else 0.02, 1.0 if base in ("g1", "g2", "gf") else 0.0)
        _normal(run.mom[k], gen, 1e-3)
    run.refresh_low_precision()
    run.x.copy_(torch.randn(run.x.shape, generator=gen, device=DEVICE))
    run.labels.copy_(torch.randint(0, net.classes, run.labels.shape, generator=gen, device=DEVICE))
    if case["mode"] == "eval":
        state["correct"] = torch.zeros(1, dtype=torch.int32, device=DEVICE)
    return state


def prepare(case, seed):
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    return (_prepare_cnn if case["kind"] == "cnn" else _prepare_vit)(case, gen)


# ---- one pass ------------------------------------------------------------------------------------------
def run(state):
    case, r = state["case"], state["run"]
    mode, vit = case["mode"], case["kind"] == "vit"
    if mode == "eval":
        s = torch.cuda.current_stream().cuda_stream
        if vit:
            cnnk_vit_eval_step(r.desc, r.buffers, state["correct"], s)
        else:
            cnnk.cnnk_eval_step(r.c_layers, len(r.layers), r.buffers, r.labels, r.loss, r.pred, state["correct"], s)
        return {"loss": r.loss, "probs": r.probs}
    if mode == "epoch":
        state["trainer"].train_batch(state["x"], state["y"], state["idx"], CNN_LR, MOMENTUM, WEIGHT_DECAY)
        return {"loss": r.loss, "param": state["param"], "mom": state["mom"], "running": state["running"]}
    r.step(VIT_LR if vit else CNN_LR, MOMENTUM, WEIGHT_DECAY)
    if vit:
        return {"loss": r.loss, "probs": r.probs, "grad": state["grad"], "param": state["param"]}
    return {"loss": r.loss, "probs": r.probs, "param": state["param"], "mom": state["mom"], "running": state["running"]}


# ---- what a pass cannot do without --------------------------------------------------------------------------
def work(case):
    """Flops: the matrix products at their true sizes.  Bytes: images, parameters (a training step reads
    and writes them and the momentum, and refreshes the bf16 copy), and in a training step the outputs of
    the matrix products, which the backward pass needs: written once, read once."""
    net, size = _net(case), 2 if case["dtype"] == "bf16" else 4
    train = case["mode"] != "eval"
    params = net.n_params()
    if case["kind"] == "cnn":
        forward, both = net.conv_flops()
        flops = both if train else forward
        images = math.prod(net.slots[0])
        kept = sum(math.prod(net.slots[L["y"]]) for L in net.layers if L["op"] == "conv")
    else:
        rows, d, m, pixels = net.batch * net.tokens, net.dim, net.mlp, net.image * net.image * 3
        linear = 2 * rows * (4 * d * d + 2 * d * m) * net.layers
        attention = 4 * rows * net.tokens * d * net.layers
        embed = 2 * net.batch * pixels * d
        flops = 3 * linear + 3.5 * attention + 2 * embed if train else linear + attention + embed
        images = net.batch * pixels
        kept = rows * (6 * d + m) * net.layers
    if train:
        return {"bytes": (images + 2 * kept) * size + params * (4 * 4 + (2 if size == 2 else 0)), "flops": flops}
    return {"bytes": images * size + params * size, "flops": flops}


def tolerance(case):
    """Four times what the path differed by with its sums in another order (other kernels, tiles and splits
    of the reductions; fp32: against the same step in 64 bits), after one and after two steps."""
    if case["dtype"] == "f32":
        return {"rel": 1e-5}
    return {"rel": 0.03, "max": 0.99}
