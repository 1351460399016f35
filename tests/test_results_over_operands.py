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


def _row(s, n=1): return [s.input("f32", (True, False)) for _ in range(n)]


# ---- an operand that several threads read the same element of: (spec, shapes, which results over which operands)

def _beside_elements():
    s = GraphSpec(2)
    x, (k,) = s.input("f32", (False, False)), _row(s)
    s.output(s.add(x, k), "f32")
    s.output(s.add(k, s.const(2.0)), "f32")
    return s, [(500, 300), (1, 300)], {1: 1}, ["tile", "tile"]


def _exchanged():
    """Either result reads what the other lies over."""
    s = GraphSpec(2)
    x, (a, b) = s.input("f32", (False, False)), _row(s, 2)
    s.output(s.add(s.add(x, a), b), "f32")
    s.output(s.add(a, s.mul(b, s.const(2.0))), "f32")
    s.output(s.sub(b, a), "f16")
    s.output(s.sub(a, b), "f32")
    return s, [(301, 700), (1, 700), (1, 700)], {0: 0, 1: 1, 3: 2}, ["tile"] * 5


def _running(rows, cols, decay, keep=True):
    """Normalisation that shifts by the running mean, which is updated; without `decay` the new mean is a value per column
    that the first pass could write."""
    s = GraphSpec(2)
    x, (r,) = s.input("f32", (False, False)), _row(s)
    mean = s.mul(s.reduce("sum", x, (0,), keep=keep), s.const(1.0 / rows))
    cen = s.sub(x, mean)
    top = s.reduce("max", s.apply("abs", cen), (0,), keep=keep)
    s.output(s.add(s.div(cen, top), r), "f32")
    s.output(s.add(s.mul(r, s.const(0.75)), s.mul(mean, s.const(0.25))) if decay else s.add(r, mean), "f32")
    return s, [(rows, cols), (1, cols)], {0: 0, 1: 1}, ["col", "col", "tile", "tile"]


def _planes():
    """Values per channel and place beside sums per channel: they vary along one of the reduced axes."""
    s = GraphSpec(3)
    x, k = s.input("f32", (False,) * 3), s.input("f32", (True, False, False))
    s.output(s.reduce("sum", s.add(x, k), (0, 2)), "f32")
    s.output(s.mul(k, s.const(0.5)), "f32")
    return s, [(40, 30, 400), (1, 30, 400)], {1: 1}, None


def _empty_batch():
    s = GraphSpec(3)
    x, k, r = s.input("f32", (False,) * 3), s.input("f32", (True, False, False)), s.input("f32", (True, True, False))
    s.output(s.add(s.add(k, s.reduce("sum", x, (0,), keep=True)), r), "f32")
    s.output(s.add(r, s.reduce("prod", s.reduce("sum", x, (0,), keep=True), (1,), keep=True)), "f32")
    return s, [(0, 70, 90), (1, 70, 90), (1, 1, 90)], {1: 2}, None


SHARED = {"beside elements": _beside_elements, "exchanged": _exchanged, "planes": _planes,
          "running": lambda: _running(500, 300, True), "running sum": lambda: _running(500, 300, False), "running, dropped axis": lambda: _running(5000, 96, False, False)}


@pytest.mark.parametrize("name", sorted(SHARED))
def test_a_shared_operand_is_overwritten_last(name):
    spec, shapes, over, want = SHARED[name]()
    expr = _plan(spec, shapes, over)
    classes, sources = _kernels(expr)
    if want: assert classes == want
    if name == "beside elements": assert expr.workspace == 0          # nothing a caller without one could not run
    # no launch writes such a result beside another output (the last stages have one output each)
    shared = sum(shapes[j] != shapes[0] for j in over.values())
    assert all("out1" not in src for src in sources[-shared:])
    # apart, the same expressions take no launch more than the results over operands cost
    assert len(_kernels(_plan(spec, shapes, {}))[0]) < len(classes)


def test_results_that_are_written_behind_all_readers_take_no_pass_more():
    # a bias gradient accumulated beside the gradient that is written over its input; a total over everything
    s = GraphSpec(2)
    x, (k,), t = s.input("f32", (False, False)), _row(s), s.input("f32", (True, True))
    y = s.apply("max", s.add(x, k), s.const(0.0))
    s.output(y, "f32")
    s.output(s.add(k, s.reduce("sum", y, (0,), keep=True)), "f32")
    for over in ({}, {0: 0, 1: 1}):
        assert _kernels(_plan(s, [(2000, 512), (1, 512), (1, 1)], over))[0] == ["col"]
    s = GraphSpec(2)
    x, t = s.input("f32", (False, False)), s.input("f32", (True, True))
    rows = s.reduce("sum", s.apply("exp", s.sub(x, s.reduce("max", x, (1,), keep=True))), (1,), keep=True)
    s.output(rows, "f32")
    s.output(s.add(t, s.reduce("sum", rows, (0,), keep=True)), "f32")
    for over in ({}, {1: 1}):
        assert _kernels(_plan(s, [(640, 3000), (1, 1)], over))[0] == ["row"]
    # an operand that no output reads is only memory
    s = GraphSpec(2)
    x, (k, b) = s.input("f32", (False, False)), _row(s, 2)
    s.output(s.add(x, b), "f32")
    s.output(s.mul(b, s.const(2.0)), "f32")
    assert _kernels(_plan(s, [(500, 300), (1, 300), (1, 300)], {1: 1}))[0] == ["tile"]


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
@pytest.mark.parametrize("name", sorted(SHARED) + ["empty batch"])
def test_results_over_a_shared_operand(name, oracle, G):
    spec, shapes, over, _ = _empty_batch() if name == "empty batch" else SHARED[name]()
    host = _inputs(spec, shapes, np.random.default_rng(5))
    print(f"[case] {name} {shapes}", flush=True)
    _, got = _run(G, spec, host, over)
    want = oracle.evaluate(spec, host, nthreads=4)
    for k, (g, w) in enumerate(zip(got, want)):
        bar = G.h.HALF if w.dtype == np.float16 else G.h.REDUCTION if name == "planes" and k == 0 else G.h.ELEMENTWISE
        G.h.compare(f"output {k}", g, w, *bar)


@pytest.mark.gpu
@pytest.mark.parametrize("rows,cols,total", PICKED)
def test_picked_elements_over_their_row(rows, cols, total, oracle, G):
    spec, shapes = _picked(rows, cols, total)
    host = _inputs(spec, shapes, np.random.default_rng(rows))
    host[0] -= np.float32(1.0)
    print(f"[case] {rows} {cols} {total}", flush=True)
    _, got = _run(G, spec, host, {0: 0})
    for k, w in enumerate(oracle.evaluate(spec, host, nthreads=4)): G.h.compare(f"output {k}", got[k], w, *G.h.ELEMENTWISE)
