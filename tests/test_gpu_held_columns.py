"""GPU parity of chained reductions down columns that a workgroup holds whole in its registers: one launch for the
statistics and the normalised tensor.  Strips whose last vector is cut, a last strip narrower than a vector, a last step that
some threads have no row for, operands read for the outputs only, results written over either operand."""
import numpy as np
import pytest

from tests.test_gpu_ops_and_layouts import G, run_spec  # noqa: F401  (G is the fixture)
from workloads import GraphSpec

pytestmark = pytest.mark.gpu


def _spec(storage, rows):
    s = GraphSpec(2)
    x = s.input(storage, (False, False))
    y = s.input(storage, (False, False))                            # for the outputs only
    gamma = s.input("f32", (True, False))
    inv = s.const(1.0 / rows)
    mean = s.mul(s.reduce("sum", x, (0,), keep=True), inv)
    cen = s.sub(x, mean)
    var = s.mul(s.reduce("sum", s.apply("sqr", cen), (0,), keep=True), inv)
    top = s.reduce("max", s.apply("abs", cen), (0,), keep=True)
    n = s.mul(cen, s.apply("recip", s.apply("sqrt", s.add(var, s.const(1e-5)))))
    s.output(s.add(s.mul(n, gamma), y), storage)
    s.output(var, "f32")
    s.output(top, "f32")
    return s


# [1024, 8]: one step a thread; [1281, 64]; [1030, 37]: a cut vector; [1200, 722], [1539, 33]: a last strip of two columns and of
# one; [2047, 300], [4096, 132], [3000, 50]: a last step that some threads have no row for
SHAPES = [(1024, 8), (1281, 64), (1030, 37), (1200, 722), (1539, 33), (2047, 300), (4096, 132), (3000, 50)]


@pytest.mark.parametrize("rows,cols", SHAPES)
@pytest.mark.parametrize("storage", ["f32", "f16"])
def test_normalisation_of_held_columns(rows, cols, storage, oracle, G):
    dt = np.float32 if storage == "f32" else np.float16
    rng = np.random.default_rng(rows + cols)
    x = (rng.standard_normal((rows, cols)) * 2 + 0.5).astype(dt)
    x[rows - 1, cols - 1] = np.nan                      # the last column only
    y = rng.standard_normal((rows, cols)).astype(dt)
    gamma = rng.uniform(0.5, 1.5, (1, cols)).astype(np.float32)
    spec = _spec(storage, rows)
    print(f"[case] {storage} {rows} {cols}", flush=True)
    expr, got = run_spec(G, spec, [x, y, gamma])
    assert expr.info()["kernel_class"] == "col" and "sm1_" in expr.source(), expr.info()
    want = oracle.evaluate(spec, [x, y, gamma], nthreads=4)
    G.h.compare("normalised", got[0], want[0], *(G.h.ELEMENTWISE if storage == "f32" else G.h.HALF))
    G.h.compare("variance", got[1], want[1], *G.h.REDUCTION)         # terms of one sign
    G.h.compare("largest deviation", got[2], want[2], *G.h.ELEMENTWISE)
    # over the input, in place
    torch = G.torch
    xd, yd, gd = (torch.from_numpy(a).cuda() for a in (x, y, gamma))
    e2 = G.ewf.Expression(spec)
    outs = [xd] + G.h.alloc_outputs(e2, spec, [xd, yd, gd])[1:]
    ws = G.h.make_workspace(e2, [xd, yd, gd], outs)
    e2.run([xd, yd, gd], outs, (), ws, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    G.h.compare("in place", outs[0].cpu().numpy(), want[0], *(G.h.ELEMENTWISE if storage == "f32" else G.h.HALF))
    # (vectors that the last column cuts belong to two threads: such calls take passes)
    assert e2.info()["kernel_class"] == ("multi" if cols % 2 else "col"), e2.info()
    # over the operand that each row's outputs read just before they are written
    xd = torch.from_numpy(x).cuda()
    e3 = G.ewf.Expression(spec)
    outs = [yd] + outs[1:]
    ws = G.h.make_workspace(e3, [xd, yd, gd], outs)
    e3.run([xd, yd, gd], outs, (), ws, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert e3.info()["kernel_class"] == ("multi" if cols % 2 else "col"), e3.info()
    G.h.compare("over the other operand", outs[0].cpu().numpy(), want[0], *(G.h.ELEMENTWISE if storage == "f32" else G.h.HALF))
