"""GPU parity of rows that end inside a vector: every number of elements the end can leave (1..7
float16, 1..3 float32), in every kernel class that reads such rows with wide accesses, with and
without the streaming hint, over an input in place, next to rows of NaN that must not leak."""
import numpy as np
import pytest

from tests.test_gpu_ops_and_layouts import G, run_spec  # noqa: F401  (G is the fixture)
from workloads import GraphSpec

pytestmark = pytest.mark.gpu


def _lnorm(storage, cols):
    s = GraphSpec(2)
    x = s.input(storage, (False, False))
    gamma, beta = s.input(storage, (True, False)), s.input(storage, (True, False))
    mean = s.mul(s.reduce("sum", x, (1,), keep=True), s.const(1.0 / cols))
    cen = s.sub(x, mean)
    var = s.mul(s.reduce("sum", s.apply("sqr", cen), (1,), keep=True), s.const(1.0 / cols))
    rstd = s.apply("recip", s.apply("sqrt", s.add(var, s.const(1e-5))))
    s.output(s.add(s.mul(s.mul(cen, rstd), gamma), beta), storage)
    return s


CUTS = [("f16", r) for r in range(1, 8)] + [("f32", r) for r in range(1, 4)]


@pytest.mark.parametrize("streaming", [0, 1])
@pytest.mark.parametrize("storage,cut", CUTS)
def test_rows_cut_inside_a_vector(storage, cut, streaming, oracle, G):
    dt, vec = (np.float16, 8) if storage == "f16" else (np.float32, 4)
    bar = G.h.HALF if storage == "f16" else G.h.REDUCTION
    rng = np.random.default_rng(cut + 10 * streaming)
    # 4 * vec + cut: the shortest row such accesses are used for; the others end in the first and in
    # a later step of a thread
    for rows, cols in ((9, 4 * vec + cut), (7, 128 * vec + cut), (5, 520 * vec + cut)):
        x = (rng.standard_normal((rows, cols)) * 2).astype(dt)
        x[1::3] = np.nan                                         # never read into a neighbouring row's result
        gb = [rng.uniform(0.5, 1.5, (1, cols)).astype(dt), rng.uniform(-0.5, 0.5, (1, cols)).astype(dt)]
        print(f"[case] layer normalisation {storage} {rows} x {cols} streaming={streaming}", flush=True)
        spec = _lnorm(storage, cols)
        expr, got = run_spec(G, spec, [x] + gb, streaming=streaming)
        assert expr.info()["kernel_class"] == "row" and expr.info()["vec"] == vec, expr.info()
        want = oracle.evaluate(spec, [x] + gb, nthreads=2)
        # the subtraction of the mean cancels: relative to |x| + |mean| over the deviation, here below 8
        G.h.compare("normalised", got[0], want[0], bar[0], 8 * bar[1])
        # the same over the input itself
        torch = G.torch
        xd, rest = torch.from_numpy(x).cuda(), [torch.from_numpy(a).cuda() for a in gb]
        e2 = G.ewf.Expression(spec, streaming=streaming)
        ws = G.h.make_workspace(e2, [xd] + rest, [xd])
        e2.run([xd] + rest, [xd], (), ws, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(xd.cpu().numpy(), got[0])

        # element-wise (float16: wide only where the strict width leaves 2-byte accesses) and reducing tiles
        print(f"[case] element-wise and sums {storage} {rows} x {cols} streaming={streaming}", flush=True)
        s = GraphSpec(2)
        a, b = s.input(storage, (False, False)), s.input(storage, (True, False))
        s.output(s.add(s.mul(a, b), s.const(0.25)), storage)
        expr, got = run_spec(G, s, [x, gb[0]], streaming=streaming)
        assert expr.info()["kernel_class"] == "tile" and ("ewf_ld_u<" in expr.source()) == (storage == "f16" and cut % 2 == 1), expr.info()
        want = oracle.evaluate(s, [x, gb[0]], nthreads=2)
        G.h.compare("scaled", got[0], want[0], *(G.h.HALF if storage == "f16" else G.h.ELEMENTWISE))
        s = GraphSpec(2)
        a, b = s.input(storage, (False, False)), s.input(storage, (False, False))
        v = s.mul(a, b)
        s.output(v, "f32")
        s.output(s.reduce("sum", v, (0, 1)), "f32")
        y = np.where(np.isnan(x), dt(1), x)
        # views with different pitches, so that the two dimensions stay apart
        wide = np.zeros((rows, cols + 3), dt); wide[:, 1:1 + cols] = y
        expr, got = run_spec(G, s, [wide[:, 1:1 + cols], y], streaming=streaming)
        assert expr.info()["kernel_class"] == "tile_reduce" and expr.info()["vec"] == vec and "ewf_ld_u<" in expr.source(), expr.info()
        want = oracle.evaluate(s, [wide[:, 1:1 + cols], y], nthreads=2)
        G.h.compare("product", got[0], want[0], *G.h.ELEMENTWISE)
        G.h.compare("sum", got[1], want[1], *G.h.REDUCTION)       # squares: terms of one sign
