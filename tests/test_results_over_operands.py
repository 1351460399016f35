"""Results written over an operand (the same pointer, shape and strides): which kernels such calls may take, on the CPU,
and their parity on the GPU.  Vectors cut by the last column belong to two threads, which may not be where one of them
still reads what the other has written."""
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


def _plan(spec, shapes, over):
    """Plans for dense tensors; `over` maps an output to the input it is written over."""
    expr = ewf.Expression(spec)
    ins = [ref(BASE + (k << 32), shape) for k, shape in enumerate(shapes)]
    outs = [ins[over[k]] if k in over else ref(BASE + (16 + k << 32), shape) for k, shape in enumerate(expr.output_shapes(ins))]
    expr.plan(ins, outs)
    return expr


def _run(G, spec, host, over):
    torch = G.torch
    dev = [torch.from_numpy(a.copy()).cuda() for a in host]
    expr = G.ewf.Expression(spec)
    outs = G.h.alloc_outputs(expr, spec, dev)
    for k, j in over.items(): outs[k] = dev[j]
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
