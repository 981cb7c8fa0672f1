"""The work whose speed counts: what a training program has this library do, through the Python entry points.

Each listed case stands for one such use (its comment in `listed` says which); `draw` gives further cases of the
same kinds with other sizes, optimizers and options.  All inputs are made on the GPU from the seed alone.

A case is a dict of plain values:
  op       step       one fused optimizer step over a parameter list
           release    the same list stepped tensor by tensor in reverse order, as a backward pass with gradient
                      release does
           step_ex    a step of the ablation / reference variants (`split`, `quant`: which technique is on)
           compress   FP32 optimizer state -> compressed layout;  decompress: the way back
           checkpoint gather the state into a blob, then scatter it into the buffers of a second list
           codec      the six standalone codecs on one array, each once
           nmse       the quantisation error of one array
  list     a parameter list of `workloads` ("odd", "flat", "resnet50", "gpt2", "llama": `layers` decoder layers with
           embedding and head, "layer": one decoder layer), or "mixed": `tensors` tensors of uneven, mostly odd sizes
           drawn from `shape`, `numel` elements in all
  kind     adamw, sgd or lion
  exact    AdamW step: flashoptim_adamw_step_exact instead of flashoptim_adamw_step
  schedule the learning rate of every tensor changes before each step
"""
import math
import random

import numpy as np
import torch

import paper_2602_23349_amd as fo
import workloads as W

HYPER = {
    "adamw": dict(lr=1e-3, wd=0.01, beta1=0.9, beta2=0.999, eps=1e-8),
    "sgd": dict(lr=1e-2, wd=5e-4, momentum=0.9),
    "lion": dict(lr=1e-4, wd=0.1, beta1=0.9, beta2=0.99),
}
FIRST_STEP = 1000          # the step counter of a program in the middle of its training
GROUP = 32


def listed():
    return [
        # a list of small tensors of every awkward size, as adapters, norms and biases give it: launch and look-up latency
        dict(name="odd_sizes_sgd", op="step", kind="sgd", list="odd"),
        # one flat buffer of 2^20 parameters (the smallest of the benchmark's workloads), bit-exact entry point
        dict(name="flat_1m_adamw", op="step", kind="adamw", list="flat", numel=1 << 20, exact=True),
        # a small vision model: 161 tensors, most of them tiny
        dict(name="resnet50_adamw", op="step", kind="adamw", list="resnet50", exact=True),
        # a small language model under a learning-rate schedule: every descriptor changes with every step
        dict(name="gpt2_lion_schedule", op="step", kind="lion", list="gpt2", schedule=True),
        # the largest: Llama-3.1-8B's embedding, head and four of its layers, rows of absent tokens without a gradient
        dict(name="llama_4l_adamw", op="step", kind="adamw", list="llama", layers=4, exact=True),
        # one decoder layer stepped by gradient release: nine calls, default entry point
        dict(name="layer_release_adamw", op="release", kind="adamw", list="layer"),
        # the plain FP32 optimizer that the compressed one is compared with, one decoder layer
        dict(name="layer_fp32_adamw", op="step_ex", kind="adamw", list="layer", split=False, quant=False),
        # adoption of the compressed layout from an FP32 checkpoint, and export to one
        dict(name="gpt2_compress", op="compress", kind="adamw", list="gpt2"),
        dict(name="gpt2_decompress", op="decompress", kind="adamw", list="gpt2"),
        # save and resume of a small model
        dict(name="resnet50_checkpoint", op="checkpoint", kind="adamw", list="resnet50"),
        # the standalone encoders and decoders on a tensor of GPT-2's embedding's size
        dict(name="codec_38m", op="codec", numel=50257 * 768),
        # quantisation error of a momentum buffer of a mid-sized matrix, as logged during a run
        dict(name="nmse_momentum_16m", op="nmse", state="momentum", linear=False, numel=4096 * 4096),
    ]


def _log_int(rng, lo, hi):
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return max(lo, min(hi, n))


def _draw_list(rng, lo, hi):
    """A flat tensor or a mixed list of lo to hi elements in all; half of the sizes are odd by chance, none is rounded."""
    n = _log_int(rng, lo, hi)
    if rng.random() < 0.3:
        return dict(list="flat", numel=n)
    return dict(list="mixed", numel=n, tensors=_log_int(rng, 2, 300), shape=rng.randrange(1 << 20))


def draw(rng):
    op = rng.choices(["step", "release", "step_ex", "compress", "decompress", "checkpoint", "codec", "nmse"],
                     weights=[10, 2, 2, 1.5, 1.5, 1.5, 1.5, 1.5])[0]
    kind = rng.choice(["adamw", "adamw", "sgd", "lion"])
    if op == "codec":
        return dict(op=op, numel=_log_int(rng, 200_000, 100_000_000))
    if op == "nmse":
        return dict(op=op, state=rng.choice(["momentum", "variance"]), linear=rng.random() < 0.5,
                    numel=_log_int(rng, 200_000, 100_000_000))
    c = dict(op=op, kind=kind)
    if op == "step":
        c.update(_draw_list(rng, 200_000, 1_500_000_000))
        c["schedule"] = rng.random() < 0.3
    elif op == "release":
        c.update(list="mixed", numel=_log_int(rng, 1_000_000, 300_000_000), tensors=_log_int(rng, 2, 40),
                 shape=rng.randrange(1 << 20))
    elif op == "step_ex":
        c.update(_draw_list(rng, 200_000, 300_000_000))
        c["split"], c["quant"] = rng.choice([(True, False), (False, True), (False, False)])
    else:
        c.update(_draw_list(rng, 200_000, 300_000_000))
    if kind == "adamw" and op in ("step", "release"):
        c["exact"] = rng.random() < 0.5
    return c


# ------------------------------------------------------------------------------- parameter lists --

def _specs(case):
    """(element count, role) of every tensor of the case's list."""
    name = case["list"]
    if name == "odd":
        specs = W.odd_sizes()
    elif name == "resnet50":
        specs = W.resnet50()
    elif name == "gpt2":
        specs = W.gpt2_small()
    elif name == "llama":
        return [(s.numel, "embedding" if s.name.startswith("embed") else s.role) for s in W.llama31_8b(case["layers"])]
    elif name == "layer":
        specs = [s for s in W.llama31_8b(1) if s.name.startswith("layers.0.")]
    elif name == "flat":
        return [(case["numel"], "matrix")]
    else:
        r = random.Random(case["shape"])
        share = [math.exp(r.uniform(0.0, 9.0)) for _ in range(case["tensors"])]
        total = sum(share)
        return [(max(1, int(case["numel"] * s / total)), r.choice(["matrix", "matrix", "gain", "bias"])) for s in share]
    return [(s.numel, s.role) for s in specs]


def _layout(specs):
    """First element of every tensor in one array that holds them all, each on a multiple of 256, and its length."""
    first, end = [], 0
    for n, _ in specs:
        first.append(end)
        end += (n + 255) // 256 * 256
    return first, end


# ------------------------------------------------------------------------------------ the inputs --

def _gen(seed, i, stream):
    g = torch.Generator(device="cuda")
    g.manual_seed(W.seed_for(seed, i, 0, stream))
    return g


def _randn(n, g):
    return torch.randn(n, dtype=torch.float32, device="cuda", generator=g)


def _grouped(x):
    """x as rows of GROUP elements, the last one filled up with zeros."""
    pad = -x.numel() % GROUP
    return (torch.nn.functional.pad(x, (0, pad)) if pad else x).view(-1, GROUP)


def _draw_tensor(n, role, i, seed):
    """What one parameter looks like in the middle of a run: FP32 theta, m, v and a BF16 gradient."""
    g = _gen(seed, i, 11)
    theta = _randn(n, g).mul_(0.02)
    if role == "gain":
        theta.add_(1.0)
    sigma = W.tensor_sigma(i, seed, 1e-5, 1e-3)
    spread = _randn(n, g).mul_(0.7).exp_().mul_(sigma)      # root of the second moment, uneven within a tensor
    grad = _randn(n, g).mul_(spread)
    m = _randn(n, g).mul_(0.25).mul_(spread)
    v = _randn(n, g).mul_(0.1).exp_().mul_(spread).mul_(spread)
    if role == "embedding":
        # rows of 4096: most tokens are absent from a batch, some have not occurred at all so far
        u = torch.rand(n // 4096, 1, device="cuda", generator=g)
        grad.view(-1, 4096).mul_((u < 0.4).float())
        for x in (m, v):
            x.view(-1, 4096).mul_((u < 0.9).float())
    return theta, m, v, grad.to(torch.bfloat16)


def _half_ulp(param):
    """Half the spacing of BF16 numbers at each element of param, in FP64."""
    e = torch.bitwise_right_shift(param.view(torch.int16).to(torch.int64), 7).bitwise_and_(0xff).clamp_(min=1)
    return e.add_(1023 - 135).bitwise_left_shift_(52).view(torch.float64)


def _encode_theta(theta):
    param = theta.to(torch.bfloat16)
    e = (theta.double() - param.double()) / _half_ulp(param)
    return param, torch.round(e.clamp_(-1.0, 1.0).mul_(127.0)).to(torch.int8)


def _scale(rows):
    s = rows.amax(1, keepdim=True).clamp_(max=65504.0).to(torch.float16)
    return s, torch.where(s == 0, torch.inf, s.float())


def _encode_m(m):
    rows = _grouped(m)
    s, d = _scale(rows.abs())
    x = rows / d
    q = torch.round((2 * x / (1 + x.abs())).mul_(127.0)).clamp_(-127, 127).to(torch.int8)
    return q.view(-1)[:m.numel()], s.view(-1)


def _encode_v(v):
    rows = _grouped(v).sqrt()
    s, d = _scale(rows)
    q = torch.round((rows / d).mul_(255.0)).clamp_(0, 255).to(torch.uint8)
    return q.view(-1)[:v.numel()], s.view(-1)


def _by_group(scale, n):
    return scale.double().repeat_interleave(GROUP)[:n]


def _decode_theta(param, rho):
    return param.double() + rho.double() / 127.0 * _half_ulp(param)


def _decode_m(q, scale):
    z = q.double() / 127.0
    return z / (2.0 - z.abs()) * _by_group(scale, q.numel())


def _decode_v(q, scale):
    return (q.double() / 255.0 * _by_group(scale, q.numel())).square_()


def _fill(case, views, specs, seed):
    """Puts the drawn values into whichever of the arrays the buffers have."""
    for i, ((n, role), b) in enumerate(zip(specs, views)):
        theta, m, v, grad = _draw_tensor(n, role, i, seed)
        if b.param is not None:
            p, r = _encode_theta(theta)
            b.param.copy_(p)
            b.rho.copy_(r)
        if b.theta is not None:
            b.theta.copy_(theta)
        if b.grad is not None:
            b.grad.copy_(grad)
        if b.m_q is not None:
            q, s = _encode_m(m)
            b.m_q.copy_(q)
            b.m_scale.copy_(s)
        if b.v_q is not None:
            q, s = _encode_v(v)
            b.v_q.copy_(q)
            b.v_scale.copy_(s)
        if b.m is not None:
            b.m.copy_(m)
        if b.v is not None:
            b.v.copy_(v)
        hp = HYPER[case["kind"]]
        b.lr, b.weight_decay = hp["lr"], (hp["wd"] if role in ("matrix", "embedding") else 0.0)


def _buffers(case, specs, **form):
    """One set of arrays for the whole list, and each tensor's part of it."""
    first, end = _layout(specs)
    arena = fo.ParamBuffers(end, case["kind"], **form)
    return arena, [arena.shard(f, n) for f, (n, _) in zip(first, specs)]


class _Both:
    """The compressed and the FP32 arrays of one tensor, as the conversions take them."""

    def __init__(self, packed, plain):
        self.flags = packed.flags
        self.numel, self.lr, self.weight_decay = packed.numel, 0.0, 0.0
        self.param, self.rho, self.grad = packed.param, packed.rho, None
        self.m_q, self.m_scale, self.v_q, self.v_scale = packed.m_q, packed.m_scale, packed.v_q, packed.v_scale
        self.theta, self.m, self.v = plain.theta, plain.m, plain.v


def _state_arrays(arena):
    return [x for x in (arena.param, arena.rho, arena.m_q, arena.m_scale, arena.v_q, arena.v_scale, arena.theta, arena.m,
                        arena.v) if x is not None]


def _draw_array(case, seed):
    theta, m, v, _ = _draw_tensor(case["numel"], "matrix", 0, seed)
    return theta, m, v


def prepare(case, seed):
    op = case["op"]
    s = dict(case=case, op=op, t=FIRST_STEP)
    if op in ("codec", "nmse"):
        n = case["numel"]
        theta, m, v = _draw_array(case, seed)
        if op == "nmse":
            s["x"] = m if case["state"] == "momentum" else v
            return s
        ng = (n + GROUP - 1) // GROUP
        empty = lambda k, dt: torch.empty(k, dtype=dt, device="cuda")
        s.update(theta=theta, m=m, v=v)
        # destinations of the encoders, then codes for the decoders and their destinations
        s["enc"] = [empty(n, torch.bfloat16), empty(n, torch.int8), empty(n, torch.int8), empty(ng, torch.float16),
                    empty(n, torch.uint8), empty(ng, torch.float16)]
        s["codes"] = [*_encode_theta(theta), *_encode_m(m), *_encode_v(v)]
        s["dec"] = [empty(n, torch.float32) for _ in range(3)]
        return s
    specs = _specs(case)
    if op in ("compress", "decompress"):
        packed, packed_views = _buffers(case, specs, with_grad=False)
        plain, plain_views = _buffers(case, specs, with_grad=False, split_weights=False, quantize_states=False)
        _fill(case, plain_views if op == "compress" else packed_views, specs, seed)
        s["list"] = fo.TensorListEx([_Both(a, b) for a, b in zip(packed_views, plain_views)], check_flags=False)
        s["out"] = _state_arrays(packed if op == "compress" else plain)
        return s
    if op == "step_ex":
        arena, views = _buffers(case, specs, split_weights=case["split"], quantize_states=case["quant"])
        _fill(case, views, specs, seed)
        s.update(list=fo.TensorListEx(views), out=_state_arrays(arena))
        return s
    arena, views = _buffers(case, specs, with_grad=op != "checkpoint")
    _fill(case, views, specs, seed)
    s.update(list=fo.TensorList(views), out=_state_arrays(arena))
    if op == "release":
        s["singles"] = [s["list"].slice(i) for i in reversed(range(len(views)))]
    if op == "checkpoint":
        other, other_views = _buffers(case, specs, with_grad=False)
        blob = torch.zeros(fo.checkpoint_size(case["kind"], [n for n, _ in specs]), dtype=torch.uint8, device="cuda")
        s.update(blob=blob, other=fo.TensorList(other_views), out=[blob] + _state_arrays(other))
    return s


def run(state):
    case, op, out = state["case"], state["op"], state.get("out")
    if op == "nmse":
        return np.array(fo.quantization_nmse(case["state"], case["linear"], state["x"]))
    if op == "codec":
        param, rho, mq, ms, vq, vs = state["enc"]
        fo.split_weights(state["theta"], param, rho)
        fo.quantize_momentum(state["m"], mq, ms)
        fo.quantize_variance(state["v"], vq, vs)
        param, rho, mq, ms, vq, vs = state["codes"]
        fo.reconstruct_weights(param, rho, state["dec"][0])
        fo.dequantize_momentum(mq, ms, state["dec"][1])
        fo.dequantize_variance(vq, vs, state["dec"][2])
        return state["enc"] + state["dec"]
    kind, hp = case["kind"], HYPER[case["kind"]]
    if op == "compress":
        fo.compress_state(kind, state["list"])
        return out
    if op == "decompress":
        fo.decompress_state(kind, state["list"])
        return out
    if op == "checkpoint":
        fo.checkpoint_pack(kind, state["list"], state["t"], state["blob"])
        return out + [fo.checkpoint_unpack(kind, state["blob"], state["other"])]
    t = state["t"] = state["t"] + 1
    if case.get("schedule"):
        lr = _scheduled_lr(hp["lr"], t)
        for i in range(state["list"].n):
            state["list"].set_hyper(i, lr=lr)
    for tensors in state["singles"] if op == "release" else (state["list"],):
        if op == "step_ex":
            if kind == "adamw":
                fo.adamw_step_ex(tensors, hp["beta1"], hp["beta2"], hp["eps"], t)
            elif kind == "sgd":
                fo.sgd_step_ex(tensors, hp["momentum"])
            else:
                fo.lion_step_ex(tensors, hp["beta1"], hp["beta2"])
        elif kind == "adamw":
            step = fo.adamw_step_exact if case.get("exact") else fo.adamw_step
            step(tensors, hp["beta1"], hp["beta2"], hp["eps"], t)
        elif kind == "sgd":
            fo.sgd_step(tensors, hp["momentum"])
        else:
            fo.lion_step(tensors, hp["beta1"], hp["beta2"])
    return out


def _scheduled_lr(base, t):
    return base * 0.5 * (1.0 + math.cos(math.pi * (t % 100_000) / 100_000))


# ------------------------------------------------------------------------- work and comparison --

def _totals(case):
    ns = [n for n, _ in _specs(case)]
    return sum(ns), sum((n + GROUP - 1) // GROUP for n in ns)


def work(case):
    """Bytes that have to be read and written, and the operations that the algorithms print per element."""
    op = case["op"]
    if op == "nmse":
        n = case["numel"]
        return {"bytes": 4 * n, "flops": 12 * n}
    if op == "codec":
        n = case["numel"]
        ng = (n + GROUP - 1) // GROUP
        return {"bytes": 2 * ((4 + 3) * n + 2 * ((4 + 1) * n + 2 * ng)), "flops": 30 * n}
    n, ng = _totals(case)
    states = 2 if case["kind"] == "adamw" else 1
    packed = 3 * n + states * (n + 2 * ng)
    plain = (1 + states) * 4 * n
    if op == "checkpoint":
        return {"bytes": 4 * packed, "flops": 0}
    if op in ("compress", "decompress"):
        return {"bytes": packed + plain, "flops": 12 * (1 + states) * n}
    split, quant = case.get("split", True), case.get("quant", True)
    state = (3 * n if split else 4 * n) + states * ((n + 2 * ng) if quant else 4 * n)
    return {"bytes": 2 * state + 2 * n, "flops": (16 * states + 10) * n}


def tolerance(case):
    """Codes, scales and weights are defined bit by bit, so a correct implementation gives the same ones.  The default
    AdamW step may round one quotient in about 10^9 the other way, which can move a weight or its correction by one
    unit; the two sums of the quantisation error are added up in FP64 in no fixed order (two runs differ by about
    1e-15)."""
    if case["op"] == "nmse":
        return {"rel": 1e-13, "max": 1e-13}
    if case.get("kind") == "adamw" and case["op"] in ("step", "release") and not case.get("exact"):
        return {"rel": 1e-6, "max": 8e-3, "differ": 1e-7}
    return "exact"


def _exact_tensor(case, n, role, i, seed):
    """FP64 results of one tensor of a step, in the order of ParamBuffers' arrays, as (elements per value, values);
    None for codes."""
    kind, hp = case["kind"], {k: float(torch.tensor(x, dtype=torch.float32)) for k, x in HYPER[case["kind"]].items()}
    split, quant = case.get("split", True), case.get("quant", True)
    theta, m, v, g = _draw_tensor(n, role, i, seed)
    theta = _decode_theta(*_encode_theta(theta)) if split else theta.double()
    m = _decode_m(*_encode_m(m)) if quant else m.double()
    g = g.double()
    t, lr = FIRST_STEP + 1, hp["lr"]
    if case.get("schedule"):
        lr = float(torch.tensor(_scheduled_lr(HYPER[kind]["lr"], t), dtype=torch.float32))
    wd = hp["wd"] if role in ("matrix", "embedding") else 0.0
    if kind == "adamw":
        v = _decode_v(*_encode_v(v)) if quant else v.double()
        m = hp["beta1"] * m + (1 - hp["beta1"]) * g
        v = hp["beta2"] * v + (1 - hp["beta2"]) * g * g
        u = (m / (1 - hp["beta1"] ** t)) / ((v / (1 - hp["beta2"] ** t)).sqrt() + hp["eps"])
    elif kind == "sgd":
        m = hp["momentum"] * m + g
        u = m
    else:
        u = torch.sign(hp["beta1"] * m + (1 - hp["beta1"]) * g)
        m = hp["beta2"] * m + (1 - hp["beta2"]) * g
    theta = theta - lr * (u + wd * theta)
    out = [(1, theta), None] if split else []
    out += [None, _top(m.abs())] if quant else []
    if kind == "adamw" and quant:
        out += [None, _top(v.sqrt())]
    out += [] if split else [(1, theta)]
    out += [] if quant else ([(1, m), (1, v)] if kind == "adamw" else [(1, m)])
    return out


def _top(x):
    return GROUP, _grouped(x).amax(1).double().clamp_(max=65504.0)


def exact(case, seed):
    op = case["op"]
    if op == "checkpoint":
        return None                     # bytes that are copied
    if op == "nmse":
        theta, m, v = _draw_array(case, seed)
        momentum = case["state"] == "momentum"
        rows = _grouped(m if momentum else v)
        x = rows.double()
        root = momentum or case["linear"]
        a = rows.abs() if root else rows.sqrt()
        s = a.amax(1, keepdim=True).clamp_(max=65504.0).to(torch.float16).double()
        d = torch.where(s == 0, torch.inf, s)
        levels = 127.0 if momentum else 255.0
        y = (x if root else x.sqrt()) / d
        if momentum and not case["linear"]:
            y = 2 * y / (1 + y.abs())
        z = torch.round(y * levels).clamp_(-levels, levels) / levels
        if momentum and not case["linear"]:
            z = z / (2 - z.abs())
        back = z * s
        if not root:
            back = back.square()
        return np.array([float((back - x).square().sum()), float(x.square().sum())])
    if op == "codec":
        theta, m, v = _draw_array(case, seed)
        enc = [theta.double(), None, None, _top(m.abs())[1], None, _top(v.double().sqrt())[1]]
        return enc + [_decode_theta(*_encode_theta(theta)), _decode_m(*_encode_m(m)), _decode_v(*_encode_v(v))]
    specs = _specs(case)
    first, end = _layout(specs)
    parts = []
    for i, (n, role) in enumerate(specs):
        if op == "compress":
            theta, m, v, _ = _draw_tensor(n, role, i, seed)
            part = [(1, theta.double()), None, None, _top(m.abs())]
            part += [None, _top(v.double().sqrt())] if case["kind"] == "adamw" else []
        elif op == "decompress":
            theta, m, v, _ = _draw_tensor(n, role, i, seed)
            part = [(1, _decode_theta(*_encode_theta(theta))), (1, _decode_m(*_encode_m(m)))]
            part += [(1, _decode_v(*_encode_v(v)))] if case["kind"] == "adamw" else []
        else:
            part = _exact_tensor(case, n, role, i, seed)
        if not parts:
            parts = [None if x is None else torch.zeros(end // x[0], dtype=torch.float64, device="cuda") for x in part]
        for whole, x in zip(parts, part):
            if x is not None:
                begin = first[i] // x[0]
                whole[begin:begin + x[1].numel()] = x[1]
    return parts
