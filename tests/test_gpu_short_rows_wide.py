"""GPU parity of short rows held by a few lanes of a wavefront: rows that end inside a vector, every
remainder, and the lane counts that wide vectors are spread over."""
import numpy as np
import pytest

from tests.test_gpu_ops_and_layouts import G, run_spec  # noqa: F401  (G is the fixture)
from workloads import GraphSpec

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage,cols", [("f32", c) for c in (17, 18, 49, 67, 143, 144, 179, 321, 999, 1001, 1023)] +
                         [("f16", c) for c in (80, 139, 257, 258, 259, 260, 261, 262, 263, 272, 288, 400, 1001, 1292, 2044)])
def test_softmax_sum_and_argmax_of_short_rows(storage, cols, oracle, G):
    dt = np.float16 if storage == "f16" else np.float32
    rng = np.random.default_rng(cols)
    rows = 4097
    x = (rng.standard_normal((rows, cols)) * 2).astype(dt)
    x[5] = np.nan                                               # never read into a neighbouring row's result
    x[7, cols - 1] = 30.0                                       # the maximum in the last element
    s = GraphSpec(2)
    xi = s.input(storage, (False, False))
    m = s.reduce("max", xi, (1,), keep=True)
    e = s.apply("exp", s.sub(xi, m))
    s.output(s.div(e, s.reduce("sum", e, (1,), keep=True)), storage)
    s.output(s.reduce("argmax", xi, (1,)), "i32")
    print(f"[case] softmax {storage} {rows} x {cols}", flush=True)
    expr, got = run_spec(G, s, [x])
    # wide accesses at any alignment: single float32 elements unless the rows are long and fit the
    # memory-side cache, float16 rows of 512 bytes and more (those that are only read keep their width)
    wide = cols % 2 == 1 and cols < 448 if storage == "f32" else cols % 8 != 0 and cols >= 256
    assert expr.info()["kernel_class"] == "lane" and ("ewf_ld_u<" in expr.source()) == wide, expr.info()
    want = oracle.evaluate(s, [x], nthreads=8)
    bar = G.h.HALF if storage == "f16" else G.h.REDUCTION
    G.h.compare("p", got[0], want[0], *bar)
    G.h.compare("argmax", got[1], want[1], 0, 0)
    assert got[1][7] == cols - 1
    s = GraphSpec(2)
    xi = s.input(storage, (False, False))
    s.output(s.reduce("sum", s.apply("abs", xi), (1,)), "f32")
    s.output(s.reduce("min", xi, (1,)), "f32")
    x[5] = 1.0
    expr, got = run_spec(G, s, [x])
    assert ("ewf_ld_u<" in expr.source()) == (storage == "f32" and cols % 2 == 1), expr.info()
    want = oracle.evaluate(s, [x], nthreads=8)
    G.h.compare("sum", got[0], want[0], *G.h.REDUCTION)          # terms of one sign
    G.h.compare("min", got[1], want[1], 0, 0)


def test_softmax_of_long_odd_rows_beyond_the_memory_side_cache(oracle, G):
    rows, cols = 25200, 1001
    x = (np.random.default_rng(1).standard_normal((rows, cols)) * 2).astype(np.float32)
    s = GraphSpec(2)
    xi = s.input("f32", (False, False))
    e = s.apply("exp", s.sub(xi, s.reduce("max", xi, (1,), keep=True)))
    s.output(s.div(e, s.reduce("sum", e, (1,), keep=True)), "f32")
    print(f"[case] softmax f32 {rows} x {cols}", flush=True)
    expr, got = run_spec(G, s, [x])
    assert expr.info()["kernel_class"] == "lane" and "ewf_ld_u<float, EWF_VEC>" in expr.source(), expr.info()
    G.h.compare("p", got[0], oracle.evaluate(s, [x], nthreads=8)[0], *G.h.REDUCTION)


@pytest.mark.parametrize("storage,cols", [("f16", 160), ("f16", 221), ("f16", 272), ("f16", 1025), ("f32", 144), ("f32", 179), ("f32", 749)])
def test_layer_normalisation_of_short_rows(storage, cols, oracle, G):
    # two levels of sums over the registers of a lane, operands that vary along the row only
    dt = np.float16 if storage == "f16" else np.float32
    rng = np.random.default_rng(cols)
    x = (rng.standard_normal((4099, cols)) * 2).astype(dt)
    gb = [rng.uniform(0.5, 1.5, (1, cols)).astype(dt), rng.uniform(-0.5, 0.5, (1, cols)).astype(dt)]
    s = GraphSpec(2)
    xi = s.input(storage, (False, False))
    ga, be = s.input(storage, (True, False)), s.input(storage, (True, False))
    cen = s.sub(xi, s.mul(s.reduce("sum", xi, (1,), keep=True), s.const(1.0 / cols)))
    var = s.mul(s.reduce("sum", s.apply("sqr", cen), (1,), keep=True), s.const(1.0 / cols))
    s.output(s.add(s.mul(s.mul(cen, s.apply("recip", s.apply("sqrt", s.add(var, s.const(1e-5))))), ga), be), storage)
    print(f"[case] layer normalisation {storage} 4099 x {cols}", flush=True)
    expr, got = run_spec(G, s, [x] + gb)
    assert expr.info()["kernel_class"] == "lane", expr.info()
    want = oracle.evaluate(s, [x] + gb, nthreads=8)
    # the subtraction of the mean cancels: relative to |x| + |mean| over the deviation, here below 8
    bar = G.h.HALF if storage == "f16" else G.h.REDUCTION
    G.h.compare("normalised", got[0], want[0], bar[0], 8 * bar[1])


@pytest.mark.parametrize("storage,rows,cols,offset,written", [("f32", 40001, 144, 0, False), ("f16", 40001, 272, 0, False), ("f32", 40001, 480, 1, False),
                                                              ("f16", 8197, 406, 0, True), ("f32", 4099, 301, 0, True), ("f32", 131, 49153, 0, True), ("f32", 131, 57341, 1, True)])
def test_sums_do_not_depend_on_what_shares_their_pass(storage, rows, cols, offset, written, G):
    """A sum and a product meet their terms in the same order, to the bit, whether or not a minimum and an
    arg-max are taken in the same pass; rows held by few lanes and long rows in registers (those are
    held by one workgroup only if they are written back)."""
    rng = np.random.default_rng(cols)
    buf = (1 + 0.01 * rng.standard_normal(rows * cols + offset)).astype(np.float16 if storage == "f16" else np.float32)
    x = buf[offset:].reshape(rows, cols)
    got = []
    for extremes in (False, True):
        s = GraphSpec(2)
        xi = s.input(storage, (False, False))
        total = s.reduce("sum", xi, (1,), keep=True)
        s.output(total, "f32")
        s.output(s.reduce("prod", xi, (1,), keep=True), "f32")
        if written:
            s.output(s.mul(xi, s.apply("recip", total)), storage)
        if extremes:
            s.output(s.reduce("min", xi, (1,)), "f32"); s.output(s.reduce("argmax", s.apply("neg", xi), (1,)), "i32")
        print(f"[case] sum and product {storage} {rows} x {cols} + {offset}, extremes {extremes}", flush=True)
        expr, out = run_spec(G, s, [x])
        assert expr.info()["kernel_class"] == ("row" if cols > 4096 else "lane") and ("part_" if cols > 4096 else "sub1_[4]") in expr.source(), expr.info()
        got.append(out)
    np.testing.assert_array_equal(got[0][0], got[1][0])
    np.testing.assert_array_equal(got[0][1], got[1][1])
    G.h.compare("sum", got[0][0], x.astype(np.float64).sum(1, keepdims=True).astype(np.float32), *G.h.REDUCTION)
    np.testing.assert_array_equal(got[1][-2], x.min(1).astype(np.float32))
    np.testing.assert_array_equal(got[1][-1], x.argmin(1).astype(np.int32))
