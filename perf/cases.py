"""The expressions this library is used for, at the sizes they meet: what its speed is measured on.

Every case describes an expression once, binds it to device tensors the way a program does that
calls it many times (`Expression`, `plan` for the workspace, `bind`), and runs it through that
prepared call.  The expressions are those of `workloads/configs.py` and, for the reductions and
row normalisations that have no workload of their own, the ones the tests evaluate.

Families and their declared ranges (`draw` spreads over all of each, odd sizes among them):

  affine    tanh(a X + b), float32, 64..4096 rows of 64..1024
  lstm      an LSTM cell's point-wise part or its backward pass, float32, batch 16..4096, hidden 128..1024
  xent      softmax cross-entropy or its gradient, float32, 128..4096 rows over 1000..65536 classes
  chansum   bias + ReLU + per-channel sums or the backward pass, float32 NCHW, 8..128 images,
            32..2048 channels, planes of 7..112 squared
  stress    the 21-operation float16 expression with a permuted operand, 1..64 images, 32..512
            channels, planes of 7..112 on a side
  bnorm     batch normalisation over the rows, float32 or float16, 1024..262144 rows of 64..4096
  lnorm     layer normalisation with scale and shift, float32 or float16, 256..65536 rows of 128..16384
  softmax   probabilities along rows, float32 or float16, 256..131072 rows of 64..16384
  axes      sums over any axes of a rank-3 tensor, float32 or float16
"""
import math

import torch

from paper_1605_02688_amd import ewf, torchmem
from workloads import GraphSpec, configs

_TORCH = {"float32": torch.float32, "float16": torch.float16, "int32": torch.int32}


def listed():
    return [
        # the smallest call: one dense layer's activation; launch latency and the call itself
        {"name": "affine_1024x256", "family": "affine", "rows": 1024, "cols": 256},
        # one training step of the large LSTM language model's cell (batch 20, 650 units: rows that
        # are no multiple of 16 bytes), four bias gradients in the same pass
        {"name": "lstm_backward_20x650", "family": "lstm", "backward": True, "batch": 20, "hidden": 650},
        # the same language model's loss over its vocabulary of ten thousand words
        {"name": "xent_1280x10000", "family": "xent", "backward": False, "rows": 1280, "vocab": 10000},
        # the gradient for a sub-word vocabulary: long rows of odd length
        {"name": "xent_backward_1280x50257", "family": "xent", "backward": True, "rows": 1280, "vocab": 50257},
        # the first layers of a convnet: large planes, the largest call
        {"name": "chansum_128x64x112x112", "family": "chansum", "backward": False, "n": 128, "c": 64, "side": 112},
        # the backward pass of its last layers: planes of 49 elements
        {"name": "chansum_backward_128x2048x7x7", "family": "chansum", "backward": True, "n": 128, "c": 2048, "side": 7},
        # many operations per element, float16, one operand channels-last
        {"name": "stress_a_64x256x56x56", "family": "stress", "reading": "A", "n": 64, "c": 256, "h": 56, "w": 56},
        # the same with the other permutation on odd planes
        {"name": "stress_b_32x192x35x35", "family": "stress", "reading": "B", "n": 32, "c": 192, "h": 35, "w": 35},
        # normalisation of activations over a batch: a plan in two passes
        {"name": "bnorm_65536x1024", "family": "bnorm", "storage": "f32", "rows": 65536, "cols": 1024},
        # normalisation of activations along their features, half-precision storage
        {"name": "lnorm_f16_8192x4096", "family": "lnorm", "storage": "f16", "rows": 8192, "cols": 4096},
        # probabilities along short rows, half-precision storage
        {"name": "softmax_f16_131072x512", "family": "softmax", "storage": "f16", "rows": 131072, "cols": 512},
        # a convnet's bias gradient: read-only sums over batch and plane
        {"name": "axes02_128x256x3136", "family": "axes", "storage": "f32", "a": 128, "b": 256, "c": 3136, "axes": "02"},
    ]


def _size(rng, lo, hi):
    """An extent of lo..hi, even over its logarithm; half of them multiples of 16 where that is
    fine enough, the others as they fall."""
    hi = max(lo, hi)
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if rng.random() < 0.5 and v >= 64:
        v = v // 16 * 16
    return min(max(v, lo), hi)


def draw(rng):
    family = rng.choice(["affine", "lstm", "xent", "chansum", "stress", "bnorm", "lnorm", "softmax", "axes"])
    case = {"family": family}
    if family == "affine":
        case.update(rows=_size(rng, 64, 4096), cols=_size(rng, 64, 1024))
    elif family == "lstm":
        case.update(backward=rng.random() < 0.5, batch=_size(rng, 16, 4096), hidden=_size(rng, 128, 1024))
    elif family == "xent":
        vocab = _size(rng, 1000, 65536)
        case.update(backward=rng.random() < 0.5, vocab=vocab, rows=_size(rng, 128, min(4096, 80_000_000 // vocab)))
    elif family == "chansum":
        backward, side, c = rng.random() < 0.5, _size(rng, 7, 112), _size(rng, 32, 2048)
        c = min(c, max(32, (64_000_000 if backward else 96_000_000) // (side * side * 8)))
        case.update(backward=backward, side=side, c=c,
                    n=_size(rng, 8, min(128, (64_000_000 if backward else 96_000_000) // (side * side * c))))
    elif family == "stress":
        h, w, c = _size(rng, 7, 112), _size(rng, 7, 112), _size(rng, 32, 512)
        case.update(reading=rng.choice("AB"), c=c, h=h, w=w, n=_size(rng, 1, min(64, 50_000_000 // (c * h * w))))
    elif family == "bnorm":
        cols = _size(rng, 64, 4096)
        case.update(storage=rng.choice(["f32", "f16"]), cols=cols, rows=_size(rng, 1024, min(262144, 67_000_000 // cols)))
    elif family == "lnorm":
        cols = _size(rng, 128, 16384)
        case.update(storage=rng.choice(["f32", "f16"]), cols=cols, rows=_size(rng, 256, min(65536, 80_000_000 // cols)))
    elif family == "softmax":
        cols = _size(rng, 64, 16384)
        case.update(storage=rng.choice(["f32", "f16"]), cols=cols, rows=_size(rng, 256, min(131072, 80_000_000 // cols)))
    else:
        b, c = _size(rng, 16, 1024), _size(rng, 16, 4096)
        case.update(storage=rng.choice(["f32", "f16"]), axes=rng.choice(["0", "1", "2", "01", "02", "12", "012"]), b=b, c=c,
                    a=_size(rng, 8, min(4096, 100_000_000 // (b * c))))
    return case


# ------------------------------------------------------------------ expressions

def _lnorm_spec(rows, cols, storage):
    s = GraphSpec(2)
    x = s.input(storage, (False, False))
    gamma, beta = s.input(storage, (True, False)), s.input(storage, (True, False))
    inv = s.const(1.0 / cols)
    mean = s.mul(s.reduce("sum", x, (1,), keep=True), inv)
    cen = s.sub(x, mean)
    var = s.mul(s.reduce("sum", s.apply("sqr", cen), (1,), keep=True), inv)
    rstd = s.apply("recip", s.apply("sqrt", s.add(var, s.const(1e-5))))
    s.output(s.add(s.mul(s.mul(cen, rstd), gamma), beta), storage)
    return s


def _softmax_spec(storage):
    s = GraphSpec(2)
    x = s.input(storage, (False, False))
    e = s.apply("exp", s.sub(x, s.reduce("max", x, (1,), keep=True)))
    s.output(s.div(e, s.reduce("sum", e, (1,), keep=True)), storage)
    return s


def _axes_spec(storage, axes):
    s = GraphSpec(3)
    s.output(s.reduce("sum", s.input(storage, (False,) * 3), axes), "f32")
    return s


def _describe(case):
    """(spec, shapes and types of the buffers, views of them, run-time scalars, bytes, outputs' names)"""
    f = case["family"]
    w = None
    if f == "affine":
        w = configs.layout_only(configs.c1_affine_tanh, rows=case["rows"], cols=case["cols"])
    elif f == "lstm":
        make = configs.c2_lstm_cell_backward if case["backward"] else configs.c2_lstm_cell
        w = configs.layout_only(make, batch=case["batch"], hidden=case["hidden"])
    elif f == "xent":
        make = configs.c3_softmax_xent_backward if case["backward"] else configs.c3_softmax_xent
        w = configs.layout_only(make, rows=case["rows"], vocab=case["vocab"])
    elif f == "chansum":
        make = configs.c4_bias_relu_chansum_backward if case["backward"] else configs.c4_bias_relu_chansum
        w = configs.layout_only(make, n=case["n"], c=case["c"], h=case["side"], w=case["side"])
    elif f == "stress":
        w = configs.layout_only(configs.c5_stress, n=case["n"], c=case["c"], h=case["h"], w=case["w"], reading=case["reading"])
    elif f == "bnorm":
        w = configs.layout_only(configs.batch_norm_axis0, rows=case["rows"], cols=case["cols"], storage=case["storage"])
    if w is not None:
        return (w.spec, [(b.shape, _TORCH[str(b.dtype)]) for b in w.buffers],
                [(v.buffer, v.shape, v.strides, v.offset) for v in w.views], list(w.scalars), w.algorithmic_bytes, w.out_names)
    st, item = case["storage"], 2 if case["storage"] == "f16" else 4
    dt = torch.float16 if st == "f16" else torch.float32
    if f == "axes":
        shape, axes = (case["a"], case["b"], case["c"]), tuple(int(d) for d in case["axes"])
        kept = math.prod(e for d, e in enumerate(shape) if d not in axes)
        return (_axes_spec(st, axes), [(shape, dt)], [(0, shape, (shape[1] * shape[2], shape[2], 1), 0)], [],
                math.prod(shape) * item + kept * 4, ["sum"])
    rows, cols = case["rows"], case["cols"]
    x = (0, (rows, cols), (cols, 1), 0)
    if f == "softmax":
        return _softmax_spec(st), [((rows, cols), dt)], [x], [], 2 * rows * cols * item, ["p"]
    row = [(k, (1, cols), (cols, 1), 0) for k in (1, 2)]
    return (_lnorm_spec(rows, cols, st), [((rows, cols), dt), ((1, cols), dt), ((1, cols), dt)], [x] + row, [],
            (2 * rows * cols + 2 * cols) * item, ["normalised"])


# ------------------------------------------------------------------ inputs

def _uniform(g, shape, lo, hi, dt):
    return torch.rand(shape, generator=g, device="cuda").mul_(hi - lo).add_(lo).to(dt)


def _normal(g, shape, mean=0.0, std=1.0, dt=torch.float32):
    return torch.randn(shape, generator=g, device="cuda").mul_(std).add_(mean).to(dt)


def _buffers(case, seed, described):
    """Device tensors from the seed: the distributions of `workloads/configs.py`."""
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    f = case["family"]
    out = []
    for k, (shape, dt) in enumerate(described):
        if dt == torch.int32:                                   # the target classes
            out.append(torch.randint(0, case["vocab"], shape, generator=g, device="cuda", dtype=torch.int32))
        elif f == "affine":
            out.append(_uniform(g, shape, -1.0, 1.0, dt))
        elif f == "stress":
            out.append(_uniform(g, shape, -2.0, 2.0, dt))
        elif f == "xent":
            out.append(_normal(g, shape, 0.0, 2.0))
        elif f == "chansum" and k in (1, 2):                    # scale, shift
            out.append(_uniform(g, shape, 0.5, 1.5, dt) if k == 1 else _uniform(g, shape, -0.5, 0.5, dt))
        elif f in ("bnorm", "axes"):
            out.append(_normal(g, shape, 0.5, 2.0, dt))
        elif f == "lnorm" and k in (1, 2):
            out.append(_uniform(g, shape, 0.5, 1.5, dt) if k == 1 else _uniform(g, shape, -0.5, 0.5, dt))
        elif f in ("lnorm", "softmax"):
            out.append(_normal(g, shape, 0.0, 2.0, dt))
        else:                                                   # lstm, chansum's activations and cotangents
            out.append(_normal(g, shape, dt=dt))
    return out


def _views(buffers, views):
    return [torch.as_strided(buffers[b].view(-1), shape, strides, offset) for b, shape, strides, offset in views]


# ------------------------------------------------------------------ the measured interface

def prepare(case, seed):
    spec, described, views, scalars, _bytes, names = _describe(case)
    buffers = _buffers(case, seed, described)
    ins = _views(buffers, views)
    expr = ewf.Expression(spec)
    outs = torchmem.alloc_outputs(expr, spec, ins)
    workspace = torchmem.make_workspace(expr, ins, outs)
    stream = torch.cuda.current_stream().cuda_stream
    state = {"case": case, "expr": expr, "ins": ins, "outs": outs, "scalars": scalars, "workspace": workspace,
             "stream": stream, "result": dict(zip(names, outs))}
    if case["family"] != "affine":
        state["call"] = expr.bind(ins, outs, scalars, workspace, stream)
    return state


def run(state):
    if "call" in state:
        state["call"].launch()                                  # a training loop's step: bound once, launched many times
    else:
        state["expr"].run(state["ins"], state["outs"], state["scalars"], state["workspace"], state["stream"])
    return state["result"]


def work(case):
    # each operand once at its own size and each output once; the operations are the scalar ones
    # of the description per element, a handful everywhere: memory bounds every case
    spec, described, _views_, _scalars, nbytes, _names = _describe(case)
    if case["family"] == "lstm" and not case["backward"]:
        elements = case["batch"] * case["hidden"]
    else:
        elements = max(math.prod(shape) for shape, _dt in described)
    return {"bytes": nbytes, "flops": elements * sum(1 for n in spec.nodes if n[0] in ("apply", "reduce"))}


def tolerance(case):
    # Relative error in the 2-norm, about four times what the evaluation shows against 64 bits over
    # these ranges: 2e-4 where results are stored as float16 (the rounding of the storage alone),
    # up to 1.5e-7 in float32, more where few terms of either sign are summed.
    if case["family"] == "stress" or case.get("storage") == "f16" and case["family"] != "axes":
        return {"rel": 1e-3, "max": 4e-3}
    return {"rel": 2e-6, "max": 4e-5}


def exact(case, seed):
    spec, described, views, scalars, _bytes, names = _describe(case)
    x = [v.double() if v.is_floating_point() else v.long() for v in _views(_buffers(case, seed, described), views)]
    f = case["family"]
    if f == "affine":
        got = [torch.tanh(scalars[0] * x[0] + x[1])]
    elif f == "lstm":
        i, f_, o = (torch.sigmoid(x[k] + x[4 + k]) for k in range(3))
        g = torch.tanh(x[3] + x[7])
        tc = torch.tanh(f_ * x[8] + i * g)
        if case["backward"]:
            dct = x[10] + x[9] * o * (1 - tc * tc)
            dz = [dct * g * i * (1 - i), dct * x[8] * f_ * (1 - f_), x[9] * tc * o * (1 - o), dct * i * (1 - g * g)]
            got = dz + [d.sum(0, keepdim=True) for d in dz] + [dct * f_]
        else:
            got = [o * tc, f_ * x[8] + i * g]
    elif f == "xent":
        m, am = x[0].max(1, keepdim=True)
        e = torch.exp(x[0] - m)
        s = e.sum(1, keepdim=True)
        if case["backward"]:
            e.div_(s)
            e.scatter_add_(1, x[1], torch.full_like(s, -1.0))
            got = [e.div_(case["rows"])]
        else:
            lsm = x[0].gather(1, x[1]) - m - torch.log(s)
            got = [m[:, 0], s[:, 0], lsm[:, 0], -lsm[:, 0], -lsm.mean(), None]
    elif f == "chansum":
        z = x[0] * x[1] + x[2]
        if case["backward"]:
            gz = (x[3] + x[4]) * (z > 0)
            del z
            got = [gz * x[1], (gz * x[0]).sum((0, 2, 3), keepdim=True), gz.sum((0, 2, 3), keepdim=True)]
        else:
            y = z.clamp_(min=0.0)
            got = [y, y.sum((0, 2, 3))]
    elif f == "stress":
        u = x[0] * x[4] + x[5]
        sp = torch.log1p(torch.exp(u))
        q = torch.pow(x[1] * x[1] + 1.0, 0.5 * x[2])
        r = torch.where(x[3] > 0, sp, q) * torch.exp(-0.5 * x[3] * x[3]) + torch.log1p(x[2] * x[2])
        got = [torch.where(x[0] > x[1], r, r * x[4] + x[5])]
    elif f == "bnorm":
        mean = x[0].mean(0, keepdim=True)
        cen = x[0] - mean
        var = (cen * cen).mean(0, keepdim=True)
        got = [cen / torch.sqrt(var + 1e-5), mean, var]
    elif f == "lnorm":
        cen = x[0] - x[0].mean(1, keepdim=True)
        got = [cen / torch.sqrt((cen * cen).mean(1, keepdim=True) + 1e-5) * x[1] + x[2]]
    elif f == "softmax":
        got = [torch.softmax(x[0], 1)]
    else:
        got = [x[0].sum(tuple(int(d) for d in case["axes"]))]
    return dict(zip(names, got))
