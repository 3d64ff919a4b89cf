"""The work that users of this library have it do, as cases that can be timed: local-block training steps of the ViT and
ResNet families on both precisions, pipelines of such blocks, and evaluation forwards, each through the calls of
include/ppll.h as paper_2411_12780_amd.binding exposes them.

A case is a flat dict: "call" (which entry point), the shape and optimizer fields of ppll_block_config under their own
names, and for a pipeline how the network is cut.  listed() holds the cases to look at, draw() gives more of the same
ranges, prepare() makes what a training program has in hand before the call, run() is one call, work() what the call
cannot do without, tolerance() how far two correct implementations at the same precision may stand apart.
"""
import math
import weakref

import torch

from paper_2411_12780_amd import binding as P
from paper_2411_12780_amd import synth

DEV = "cuda"
STEP, PIPELINE, EVAL = "step", "pipeline", "eval"
SIZES = ("arch", "precision", "input_kind", "batch", "img_h", "img_w", "img_c", "patch", "tokens", "dim", "heads", "mlp_dim",
         "depth", "aux_depth", "channels", "height", "width", "n_basic_blocks", "aux_channels", "transition_block",
         "optimizer", "momentum", "nesterov", "weight_decay", "lr", "num_classes")


def _case(name, call, wl, **more):
    c = {"name": name, "call": call}
    c.update({k: wl[k] for k in SIZES if k in wl})
    c.update(more)
    return c


def listed():
    w = synth.workload
    return [
        # the smallest step: a 64-wide ViT block on 8 images in fp32, as used to check an installation and to debug with;
        # some fifty tiny launches, so launch latency and the depth of the dependent chain count
        _case("vit tiny fp32", STEP, w("vit_tiny_fp32")),
        # the ordinary training step: one of four blocks of a 12-layer ViT on 128 images of 32 x 32
        _case("vit stage", STEP, w("vit_stage_bf16")),
        # the same stage further down the network (token activations in), on the last batch of an epoch: 50000 images
        # leave 80 for it; two auxiliary layers
        _case("vit stage last batch", STEP, w("vit_stage_act_bf16", batch=80, aux_depth=2)),
        # larger images: 96 x 96, 145 tokens
        _case("vit large image", STEP, w("vit_large_image_bf16")),
        # wide and short: 5 tokens of width 768, where reading weights costs more than multiplying by them
        _case("vit wide short", STEP, w("vit_base_paper_bf16")),
        # the largest step: 197 tokens of width 768, 128 images
        _case("vit wide long", STEP, w("vit_base_224_bf16")),
        # convolution stage at a small batch: many short launches
        _case("resnet stage", STEP, w("resnet_stage_bf16")),
        # first stage of ResNet-32 at its training batch: stem and 16 channels on 32 x 32 maps, bound by memory
        _case("resnet32 first stage", STEP, w("resnet32_stage1_bf16")),
        # third stage (64 channels on 8 x 8 maps behind a downsampling block) on the last batch of an epoch:
        # 50000 images leave 848 of 1024
        _case("resnet32 third stage tail", STEP, w("resnet32_stage3_bf16", batch=848)),
        # the whole 12-layer ViT as four blocks on four streams, one batch entering the pipeline
        _case("vit pipeline of 4", PIPELINE, w("vit_stage_bf16"), blocks=4),
        # ResNet-32 cut into eight modules on eight streams
        _case("resnet32 pipeline of 8", PIPELINE, w("resnet32_stage1_bf16"), blocks=8),
        # taking accuracies: the last block of the ViT in evaluation mode, with class scores
        _case("vit eval", EVAL, w("vit_stage_act_bf16")),
    ]


LARGEST_FLOPS = 3.7e12     # a little above the largest listed case
LARGEST_PASSES = 5.7e9     # layer inputs and outputs of the largest listed ResNet pipeline, in elements (see _map_elements)


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_vit(rng, call):
    img, patch = rng.choice(((32, 4), (32, 8), (32, 16), (64, 8), (96, 8), (96, 16), (224, 16)))
    dim = rng.choice((192, 384, 384, 768))
    wl = synth.workload("vit_stage_bf16", img_h=img, img_w=img, patch=patch, tokens=(img // patch) ** 2 + 1, dim=dim,
                        heads=dim // 64, mlp_dim=4 * dim, batch=_log(rng, 4, 128), depth=rng.randint(1, 3),
                        aux_depth=rng.randint(0, 4), input_kind=rng.choice((synth.IMAGE, synth.ACTIVATION)))
    if rng.random() < 0.5:
        wl.update(optimizer=synth.SGD, momentum=0.9, nesterov=1, weight_decay=1e-4, lr=0.01)
    return _case("", call, wl)


def _draw_vit_fp32(rng):
    img, patch = rng.choice(((32, 4), (32, 8), (32, 16), (64, 8)))
    heads = rng.choice((2, 3, 4, 6))
    dim = heads * rng.choice((16, 32, 64))
    wl = synth.workload("vit_tiny_fp32", img_h=img, img_w=img, patch=patch, tokens=(img // patch) ** 2 + 1, dim=dim, heads=heads,
                        mlp_dim=rng.choice((2, 4)) * dim, batch=_log(rng, 3, 24), depth=rng.randint(1, 3),
                        aux_depth=rng.randint(0, 1), momentum=rng.choice((0.0, 0.9)))
    return _case("", STEP, wl)


def _draw_resnet(rng, call):
    group = rng.randint(0, 2)
    wl = synth.workload("resnet32_stage%d_bf16" % (group + 1), batch=_log(rng, 24, 1024), n_basic_blocks=rng.randint(1, 5))
    if rng.random() < 0.5:      # a module in the middle of a group: neither stem nor downsampling block
        wl.update(input_kind=synth.ACTIVATION, transition_block=0)
    return _case("", call, wl)


def draw(rng):
    while True:
        kind = rng.random()
        if kind < 0.40:
            c = _draw_vit(rng, STEP)
        elif kind < 0.50:
            c = _draw_vit_fp32(rng)
        elif kind < 0.70:
            c = _draw_resnet(rng, STEP)
        elif kind < 0.80:
            c = _draw_vit(rng, EVAL)
        elif kind < 0.86:
            c = _draw_resnet(rng, EVAL)
        elif kind < 0.94:
            c = dict(_draw_vit(rng, PIPELINE), input_kind=synth.IMAGE, blocks=rng.randint(2, 4))
        else:
            c = _case("", PIPELINE, synth.workload("resnet32_stage1_bf16", batch=_log(rng, 64, 1024)), blocks=rng.randint(2, 8))
        del c["name"]
        if work(c)["flops"] <= LARGEST_FLOPS and _map_elements(c) <= LARGEST_PASSES:
            return c


# ---------------------------------------------------------------- the blocks of a case and their parameters
def _blocks(case):
    """The workload dict of every block of the case, first to last."""
    wl = dict({"momentum": 0.0, "nesterov": 0, "weight_decay": 0.0, "transition_block": 0}, **{k: case[k] for k in SIZES if k in case})
    n = case.get("blocks", 1)
    if case["call"] != PIPELINE:
        return [wl]
    if wl["arch"] == synth.VIT:
        return [dict(wl, input_kind=wl["input_kind"] if j == 0 else synth.ACTIVATION) for j in range(n)]
    return synth.resnet32_modules(n, batch=wl["batch"])


def _spec(wl):
    """(name, shape) of every parameter tensor in the order of the parameter blob."""
    s = []
    if wl["arch"] == synth.VIT:
        D, F, C = wl["dim"], wl["mlp_dim"], wl["num_classes"]
        if wl["input_kind"] == synth.IMAGE:
            s += [("pe.w", (wl["patch"] ** 2 * wl["img_c"], D)), ("pe.b", (D,)), ("cls", (D,)), ("pos", (wl["tokens"], D))]
        for l in range(wl["depth"] + wl["aux_depth"]):
            s += [("ln1.g", (D,)), ("ln1.b", (D,)), ("qkv.w", (D, 3 * D)), ("qkv.b", (3 * D,)), ("proj.w", (D, D)), ("proj.b", (D,)),
                  ("ln2.g", (D,)), ("ln2.b", (D,)), ("fc1.w", (D, F)), ("fc1.b", (F,)), ("fc2.w", (F, D)), ("fc2.b", (D,))]
        return s + [("ln.g", (D,)), ("ln.b", (D,)), ("head.w", (D, C)), ("head.b", (C,))]
    t, C, A = wl["transition_block"] - 1, wl["channels"], wl["aux_channels"]
    ci = C // 2 if t >= 0 else C
    if wl["input_kind"] == synth.IMAGE:
        s += [("stem.conv", (9, wl["img_c"], ci)), ("stem.bn.g", (ci,)), ("stem.bn.b", (ci,))]
    for i in range(wl["n_basic_blocks"]):
        co = C if t < 0 or i >= t else C // 2
        k = "0" if i == 0 else "n"
        s += [("conv1", (9, ci, co)), ("bn1.g", (co,)), ("bn1.b", (co,)), ("conv2", (9, co, co)), (k + "bn2.g", (co,)), (k + "bn2.b", (co,))]
        ci = co
    return s + [("aux.conv", (9, C, A)), ("aux.bn.g", (A,)), ("aux.bn.b", (A,)), ("head.w", (A, wl["num_classes"])), ("head.b", (wl["num_classes"],))]


def _params(wl, gen):
    """Initial parameters as the library draws them itself (weights N(0, 0.02^2), convolutions N(0, 2 / (9 Cin)), biases 0,
    norm scales 1), except that BatchNorm scales and shifts have the spread that training gives them: with shifts of 0
    every ReLU input is centred on 0, whether an input passes then hangs on the last bit of a bf16 value for one in a few
    hundred of them, and the gradients of two correct implementations stand 1 % to 4 % apart after ten such layers (0.1 %
    to 0.2 % with these shifts)."""
    parts = []
    for name, shape in _spec(wl):
        n = math.prod(shape)
        norm, leaf = "ln" in name or "bn" in name, name.split(".")[-1]
        if "conv" in name:
            v = torch.randn(n, generator=gen, device=DEV) * math.sqrt(2.0 / (9.0 * shape[1]))
        elif norm and leaf == "g":
            v = torch.full((n,), 0.35 if name == "nbn2.g" else 1.0, device=DEV)
        elif "bn" in name:
            v = torch.full((n,), 0.2 if name == "nbn2.b" else 2.0, device=DEV)
            if name == "bn1.b":
                v[1::2] = -2.0
        elif leaf == "b":
            v = torch.zeros(n, device=DEV)
        else:
            v = torch.randn(n, generator=gen, device=DEV) * 0.02
        parts.append(v)
    return torch.cat(parts)


def _find(ws, blk, kind, floats, restore):
    """View of the `floats` values of one kind (parameters, gradients, moments, BatchNorm statistics) of a block inside its
    workspace, where a training program reads them on the device.  The place is found through the public calls: a probe is
    written to the first tensor of the kind, looked for in the workspace, and taken back."""
    _, n = P.ppll_block_tensor_info(blk, kind, 0)
    probe = torch.linspace(1.2345678, 2.3456789, n)
    P.ppll_block_write_tensor(blk, kind, 0, probe.numpy())
    words = ws.view(torch.float32)
    at = None
    for row in (words[::64] == float(probe[0])).nonzero().flatten().tolist():
        if torch.equal(words[64 * row:64 * row + n].cpu(), probe):
            at = 64 * row
    P.ppll_block_write_tensor(blk, kind, 0, restore[:n].cpu().numpy())
    if at is None:
        raise RuntimeError("tensor kind %d is not in the workspace" % kind)
    return words[at:at + floats]


class _State:
    """What a training program holds: the workspace, the handle, one batch on the device, output buffers."""

    def __init__(self, case):
        self.call = case["call"]
        self.blk = self.pipe = None
        # the rate that the cosine schedule gives nine tenths through training
        self.lr = synth.cosine_lr(90, 100, case["lr"])


def _state_views(ws, blk, wl, blob):
    """Gradients and updated state of a block as tensors on the device."""
    n = blob.numel()
    zeros = torch.zeros(n, device=DEV)
    views = {"params": _find(ws, blk, P.T_PARAM, n, blob), "grads": _find(ws, blk, P.T_GRAD, n, zeros),
             "moment1": _find(ws, blk, P.T_MOMENT1, n, zeros)}
    if wl["optimizer"] == synth.ADAMW:
        views["moment2"] = _find(ws, blk, P.T_MOMENT2, n, zeros)
    if wl["arch"] == synth.RESNET:
        channels = sum(shape[0] for name, shape in _spec(wl) if "bn" in name and name.endswith(".g"))
        views["bn_mean"] = _find(ws, blk, P.T_BN_MEAN, channels, zeros)
        views["bn_var"] = _find(ws, blk, P.T_BN_VAR, channels, torch.ones(channels))
    return views


def prepare(case, seed):
    wls = _blocks(case)
    first, last = wls[0], wls[-1]
    dtype = torch.bfloat16 if first["precision"] == synth.BF16 else torch.float32
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))
    blobs = [_params(wl, gen) for wl in wls]
    s = _State(case)
    # images normalised to mean 0 and deviation 1 (or activations of that scale), labels uniform
    s.x = torch.randn(synth.input_shape(first), generator=gen, device=DEV).to(dtype)
    s.y = torch.randint(0, first["num_classes"], (first["batch"],), generator=gen, device=DEV, dtype=torch.int32)
    cfgs = [P.make_config(wl) for wl in wls]
    if case["call"] == PIPELINE:
        depth = 2
        nbytes = P.ppll_pipeline_workspace_bytes(cfgs, depth)
        s.ws = torch.empty(nbytes, dtype=torch.uint8, device=DEV)
        s.streams = [torch.cuda.Stream() for _ in cfgs]
        torch.cuda.synchronize()
        s.pipe = P.ppll_pipeline_init(cfgs, depth, s.ws, nbytes, [q.cuda_stream for q in s.streams], [b.cpu().numpy() for b in blobs])
        weakref.finalize(s, P.ppll_pipeline_destroy, s.pipe)
        s.losses = torch.zeros(len(cfgs), device=DEV)
        addr, size = P.ppll_pipeline_output(s.pipe)
        at = addr - s.ws.data_ptr()
        s.out = {"x_out": s.ws[at:at + size].view(dtype), "losses": s.losses}
        for j, (wl, b) in enumerate(zip(wls, blobs)):
            for k, v in _state_views(s.ws, P.ppll_pipeline_block(s.pipe, j), wl, b).items():
                s.out["block%d.%s" % (j, k)] = v
        return s
    nbytes = P.ppll_block_workspace_bytes(cfgs[0])
    s.ws = torch.empty(nbytes, dtype=torch.uint8, device=DEV)
    s.blk = P.ppll_block_init(cfgs[0], s.ws, nbytes, blobs[0].cpu().numpy(), None)
    weakref.finalize(s, P.ppll_block_destroy, s.blk)
    s.x_out = torch.empty(synth.output_shape(last), dtype=dtype, device=DEV)
    if case["call"] == EVAL:
        s.logits = torch.zeros(last["batch"], last["num_classes"], device=DEV)
        s.out = {"x_out": s.x_out, "logits": s.logits}
    else:
        s.loss = torch.zeros(1, device=DEV)
        s.out = dict({"x_out": s.x_out, "loss": s.loss}, **_state_views(s.ws, s.blk, first, blobs[0]))
    return s


def run(s):
    if s.pipe is not None:
        P.ppll_pipeline_step(s.pipe, s.x, s.y, s.lr, s.losses)
    elif s.call == EVAL:
        P.ppll_block_forward_eval(s.blk, s.x, s.x_out, s.logits, torch.cuda.current_stream().cuda_stream)
    else:
        P.ppll_block_step(s.blk, s.x, s.y, s.lr, s.x_out, s.loss, torch.cuda.current_stream().cuda_stream)
    return s.out


# ---------------------------------------------------------------- what a call cannot do without
def _vit_flops(wl, train):
    """Contractions of one pass (multiply-add = 2): forward, input gradients, weight gradients; of the last auxiliary layer
    keys and values for every token and the rest for the class token alone, since the head reads no other row."""
    B, T, D, F = wl["batch"], wl["tokens"], wl["dim"], wl["mlp_dim"]
    M, times = B * T, 3.0 if train else 1.0
    layer = 2.0 * M * (4 * D * D + 2 * D * F) + 4.0 * B * T * T * D
    cls = 2.0 * M * 2 * D * D + 2.0 * B * (2 * D * D + 2 * D * F) + 4.0 * B * T * D
    total = times * layer * wl["depth"]
    if wl["aux_depth"]:
        total += times * (layer * (wl["aux_depth"] - 1) + cls)
    total += times * 2.0 * B * D * wl["num_classes"]
    if wl["input_kind"] == synth.IMAGE:     # the image needs no gradient
        total += (2.0 if train else 1.0) * 2.0 * B * (T - 1) * wl["patch"] ** 2 * wl["img_c"] * D
    return total


def _convs(wl):
    """(output pixels, Cin, Cout, whether its input needs a gradient) of every convolution."""
    B, C, H, W, t = wl["batch"], wl["channels"], wl["height"], wl["width"], wl["transition_block"] - 1
    m = 2 if t >= 0 else 1
    stem, ci = wl["input_kind"] == synth.IMAGE, C // m
    out = [(B * m * H * m * W, wl["img_c"], ci, False)] if stem else []
    for i in range(wl["n_basic_blocks"]):
        co, px = (ci, B * m * H * m * W) if i < t else (C, B * H * W)
        out += [(px, ci, co, stem or i > 0), (px, co, co, True)]
        ci = co
    return out + [(B * ((H + 1) // 2) * ((W + 1) // 2), C, wl["aux_channels"], True)]


def _map_elements(case):
    """Elements that the convolutions of a ResNet case read and write, over forward and backward: what such a case costs."""
    return sum(px * (ci + co) * (1.0 if case["call"] == EVAL else 3.0) for wl in _blocks(case) if wl["arch"] == synth.RESNET
               for px, ci, co, _ in _convs(wl))


def _resnet_flops(wl, train):
    total = sum(2.0 * 9 * px * ci * co * ((3 if grad else 2) if train else 1) for px, ci, co, grad in _convs(wl))
    return total + (3.0 if train else 1.0) * 2.0 * wl["batch"] * wl["aux_channels"] * wl["num_classes"]


def work(case):
    """Contractions; and every input (batch, labels, parameters, moments) read once, every output (activation, loss,
    gradients, updated parameters and moments) written once.  What passes between the layers is not counted."""
    train, total = case["call"] != EVAL, {"bytes": 0.0, "flops": 0.0}
    wls = _blocks(case)
    esz = 2 if wls[0]["precision"] == synth.BF16 else 4
    for j, wl in enumerate(wls):
        total["flops"] += (_vit_flops if wl["arch"] == synth.VIT else _resnet_flops)(wl, train)
        n = sum(math.prod(shape) for _, shape in _spec(wl))
        if j == 0:
            total["bytes"] += math.prod(synth.input_shape(wl)) * esz + 4 * wl["batch"]
        total["bytes"] += math.prod(synth.output_shape(wl)) * esz
        if train:   # parameters and moments in and out, gradients out
            total["bytes"] += 4.0 * n * (7 if wl["optimizer"] == synth.ADAMW else 5) + 4
        else:       # evaluation reads the precision the contractions take
            total["bytes"] += esz * n + 4.0 * wl["batch"] * wl["num_classes"]
    return total


def tolerance(case):
    """fp32: sums over at most a few thousand terms through up to a dozen layers.  bf16: every tensor that passes between
    layers is rounded to 8 bits of significand (2^-9 each), forward and backward; evaluation has the forward alone.  All
    gradients of a block are one output, whose tensors differ in scale: a single value may be off by most of its rms."""
    if case["precision"] == synth.FP32:
        return {"rel": 3e-5}
    return {"rel": 1e-2} if case["call"] == EVAL else {"rel": 2e-2, "max": 0.9}
