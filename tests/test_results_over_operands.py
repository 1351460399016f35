"""Results written over an operand (the same pointer, shape and strides): which kernels such calls may take, on the CPU,
and their parity on the GPU.  Vectors cut by the last column belong to two threads, and an operand that does not vary along
every axis is read by many: neither may be where one of them still reads what another has written."""
import numpy as np
import pytest

from paper_1605_02688_amd import ewf
from tests.test_gpu_ops_and_layouts import G  # noqa: F401  (the fixture)
from tests.test_host_library import BASE, ref
from workloads import GraphSpec


def _column_sums(shape, axis, storage):
    """k + sum(x) along the axis: a bias gradient that is accumulated."""
    s = GraphSpec(len(shape))
    x = s.input(storage, (False,) * len(shape))
    k = s.input("f32", tuple(d == axis for d in range(len(shape))))
    s.output(s.add(k, s.reduce("sum", x, (axis,), keep=True)), "f32")
    return s


def _normalised(rows, storage, running):
    """x less its mean per column, over the largest deviation; and the running mean, where there is one."""
    s = GraphSpec(2)
    x = s.input(storage, (False, False))
    r = s.input("f32", (True, False)) if running else None
    mean = s.mul(s.reduce("sum", x, (0,), keep=True), s.const(1.0 / rows))
    cen = s.sub(x, mean)
    s.output(s.div(cen, s.reduce("max", s.apply("abs", cen), (0,), keep=True)), storage)
    if running: s.output(s.add(s.mul(r, s.const(0.75)), s.mul(mean, s.const(0.25))), "f32")
    return s


def _plan(spec, shapes, over, **opts):
    """Plans for dense tensors; `over` maps an output to the input it is written over."""
    expr = ewf.Expression(spec, **opts)
    ins = [ref(BASE + (k << 32), shape) for k, shape in enumerate(shapes)]
    outs = [ref(BASE + ((over[k] if k in over else 16 + k) << 32), shape) for k, shape in enumerate(expr.output_shapes(ins))]
    expr.workspace = expr.plan(ins, outs)
    return expr


def _kernels(expr):
    """The kernel classes of a plan's launches, and the source of each."""
    info = expr.info()
    if info["kernel_class"] != "multi": return [info["kernel_class"]], [expr.source()]
    stages = range(info["grid_blocks"])
    return [ewf.debug_plan_info(expr.handle, k)["kernel_class"] for k in stages], [ewf.debug_source(expr.handle, k) for k in stages]


def _run(G, spec, host, over):
    torch = G.torch
    dev = [torch.from_numpy(a.copy()).cuda() for a in host]
    expr = G.ewf.Expression(spec)
    outs = G.h.alloc_outputs(expr, spec, dev)
    for k, j in over.items(): outs[k] = dev[j].view(outs[k].shape)
    ws = G.h.make_workspace(expr, dev, outs)
    expr.run(dev, outs, (), ws, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    return expr, [o.cpu().numpy() for o in outs]


def _cut(expr):
    return "ewf_ld_u<" in expr.source().split('extern "C"')[1]


SUMS = [((128, 64, 253), 1, "f32"), ((128, 64, 253), 1, "f16"), ((300, 70, 189), 1, "f16"), ((500, 129, 189), 1, "f16")]
# a last strip of one column, which the strip before holds too; [1024, 8192], [2047, 300]: whole vectors
HELD = [(1024, 8193, "f32"), (2000, 4097, "f32"), (1539, 33, "f32"), (1539, 33, "f16"), (1024, 8192, "f32"), (2047, 300, "f16")]


@pytest.mark.parametrize("shape,axis,storage", SUMS)
def test_sums_over_an_operand_keep_to_their_columns(shape, axis, storage):
    spec, shapes = _column_sums(shape, axis, storage), [shape, tuple(1 if d == axis else e for d, e in enumerate(shape))]
    assert _cut(_plan(spec, shapes, {}))
    assert not _cut(_plan(spec, shapes, {0: 1}))
    # one executable, both calls, in either order
    expr = ewf.Expression(spec)
    ins = [ref(BASE + (k << 32), s) for k, s in enumerate(shapes)]
    for out, cut in ((ins[1], False), (ref(BASE + (16 << 32), shapes[1]), True), (ins[1], False)):
        expr.plan(ins, [out])
        assert _cut(expr) == cut


@pytest.mark.parametrize("rows,cols,storage", HELD)
@pytest.mark.parametrize("running", [False, True])
def test_held_columns_over_an_operand_keep_to_their_columns(rows, cols, storage, running):
    spec, shapes = _normalised(rows, storage, running), [(rows, cols)] + [(1, cols)] * running
    held = lambda expr: "sm1_" in expr.source()
    assert held(_plan(spec, shapes, {}))
    for over in [{0: 0}] + [{1: 1}, {0: 0, 1: 1}] * running:
        assert held(_plan(spec, shapes, over)) == (cols % 2 == 0), over


def _picked(rows, cols, total):
    """One element of a row, chosen by an index, beside a result of the row's length."""
    s = GraphSpec(2)
    x, t = s.input("f32", (False, False)), s.input("i32", (False, True))
    one = s.reduce("sum", s.apply("where", s.apply("eq", s.iota(1), t), x, s.const(0.0)), (1,), keep=True)
    if total:
        s.output(s.apply("max", x, s.const(0.0)), "f32")
        s.output(s.add(one, s.reduce("max", x, (1,), keep=True)), "f32")
    else:
        s.output(s.sub(x, one), "f32")
    return s, [(rows, cols), (rows, 1)]


PICKED = [(40, 30000, True), (600, 3000, True), (600, 3000, False), (300, 20011, False), (5000, 500, False)]


@pytest.mark.parametrize("rows,cols,total", PICKED)
def test_an_element_is_not_picked_from_a_row_that_is_gone(rows, cols, total):
    spec, shapes = _picked(rows, cols, total)
    picks = lambda expr: [src for src in _kernels(expr)[1] if "const bool in_ = " in src]
    apart, over = _plan(spec, shapes, {}), _plan(spec, shapes, {0: 0})
    assert picks(apart)
    # (a wavefront's loads come before its stores, and a workgroup's before a fold that the stores wait for)
    assert not picks(over) or over.info()["kernel_class"] == "lane" or (total and over.info()["kernel_class"] == "row")


@pytest.mark.gpu
@pytest.mark.parametrize("shape,axis,storage", SUMS)
def test_sums_over_an_operand(shape, axis, storage, oracle, G):
    rng = np.random.default_rng(sum(shape))
    x = rng.uniform(0.5, 1.5, shape).astype(np.float32 if storage == "f32" else np.float16)
    k = rng.uniform(0.5, 1.5, [1 if d == axis else e for d, e in enumerate(shape)]).astype(np.float32)
    spec = _column_sums(shape, axis, storage)
    print(f"[case] {storage} {shape}", flush=True)
    _, got = _run(G, spec, [x, k], {0: 1})
    G.h.compare("sum", got[0], oracle.evaluate(spec, [x, k], nthreads=4)[0], *G.h.REDUCTION)     # terms of one sign


@pytest.mark.gpu
@pytest.mark.parametrize("rows,cols,storage", HELD)
def test_normalisation_over_its_input(rows, cols, storage, oracle, G):
    rng = np.random.default_rng(rows + cols)
    x = (rng.standard_normal((rows, cols)) * 2 + 0.5).astype(np.float32 if storage == "f32" else np.float16)
    spec = _normalised(rows, storage, False)
    print(f"[case] {storage} {rows} {cols}", flush=True)
    _, got = _run(G, spec, [x], {0: 0})
    G.h.compare("normalised", got[0], oracle.evaluate(spec, [x], nthreads=4)[0], *(G.h.ELEMENTWISE if storage == "f32" else G.h.HALF))


def _inputs(spec, shapes, rng):
    out = []
    kinds = [n[2] for n in spec.nodes if n[0] == "input"]
    for storage, shape in zip(kinds, shapes):
        if storage == "i32": out.append(rng.integers(0, shapes[0][1], shape).astype(np.int32))
        else: out.append(rng.uniform(0.5, 1.5, shape).astype(np.float32))
    return out


@pytest.mark.gpu
@pytest.mark.parametrize("rows,cols,total", PICKED)
def test_picked_elements_over_their_row(rows, cols, total, oracle, G):
    spec, shapes = _picked(rows, cols, total)
    host = _inputs(spec, shapes, np.random.default_rng(rows))
    host[0] -= np.float32(1.0)
    print(f"[case] {rows} {cols} {total}", flush=True)
    _, got = _run(G, spec, host, {0: 0})
    for k, w in enumerate(oracle.evaluate(spec, host, nthreads=4)): G.h.compare(f"output {k}", got[k], w, *G.h.ELEMENTWISE)
