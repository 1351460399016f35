"""GPU parity of column kernels at the edges of their splits: whole columns in one workgroup of 256 to
1024 threads, the first sizes that take partial results instead, narrow strips, and odd widths."""
import numpy as np
import pytest

from tests.test_gpu_ops_and_layouts import G, _moments_spec, run_spec  # noqa: F401  (G is the fixture)
from workloads import GraphSpec, configs as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,hidden", [(17, 33), (65, 130), (115, 464), (129, 512), (157, 537), (300, 208), (700, 350), (912, 1008), (2100, 36)])
def test_lstm_backward_over_the_batch(batch, hidden, oracle, G):
    w = wl.c2_lstm_cell_backward(batch=batch, hidden=hidden)
    print(f"[case] lstm backward {batch} x {hidden}", flush=True)
    expr, got = G.h.run_gpu(w)
    assert expr.info()["kernel_class"] == "col" and ("ewf_finish(" in expr.source()) == (batch >= 300), expr.info()
    want = dict(zip(w.out_names, oracle.evaluate(w.oracle_spec or w.spec, wl.host_inputs(w), w.scalars, nthreads=8)))
    for name, g, (rtol, atol) in zip(w.out_names, got, w.tol):
        # A bias gradient sums `batch` gate gradients of either sign: a tree of at most 12 levels over
        # chains of a few terms rounds by less than 24 * 2^-24 = 1.5e-6 of the sum of their
        # magnitudes, plus what the terms themselves carry (the element-wise bar, 2e-6 of each); what
        # they cancel to does not enter.
        scale = np.abs(want[name.replace("dbias", "dz")].astype(np.float64)).sum(0, keepdims=True) if name.startswith("dbias") else None
        G.h.compare(name, g, want[name], rtol, atol, scale=scale)


@pytest.mark.parametrize("storage", ["f32", "f16"])
@pytest.mark.parametrize("shape,axes", [((60, 10000), (0,)), ((1000, 2000), (0,)), ((3000, 16), (0,)), ((3001, 17), (0,)), ((12289, 4), (0,)),
                                        ((40, 1000, 64), (1,)), ((7, 513, 96), (1,)), ((257, 63), (0,))])
def test_sums_and_extremes_down_columns(shape, axes, storage, oracle, G):
    dt = np.float16 if storage == "f16" else np.float32
    rng = np.random.default_rng(shape[0] + len(shape))
    x = (rng.standard_normal(shape) * 2).astype(dt)
    x.reshape(-1)[x.size // 3] = np.nan
    s = GraphSpec(len(shape))
    v = s.input(storage, (False,) * len(shape))
    s.output(s.reduce("sum", s.apply("abs", v), axes), "f32")
    s.output(s.reduce("max", v, axes), "f32")
    s.output(s.reduce("argmax", v, axes), "i32")
    print(f"[case] columns {storage} {shape} {axes}", flush=True)
    expr, got = run_spec(G, s, [x])
    whole = shape in ((60, 10000), (7, 513, 96), (257, 63))     # columns in one workgroup each
    assert expr.info()["kernel_class"] == "col" and ("ewf_finish(" in expr.source()) == (not whole), expr.info()
    want = oracle.evaluate(s, [x], nthreads=4)
    G.h.compare("sum", got[0], want[0], *G.h.REDUCTION)          # terms of one sign
    np.testing.assert_array_equal(got[1], want[1])
    np.testing.assert_array_equal(got[2], want[2])


@pytest.mark.parametrize("shape,axes", [((2048, 8192), (0,)), ((65536, 64), (0,)), ((200, 2000), (0,)), ((5, 4096), (0,)), ((33, 7, 640), (0,)), ((3, 300000), (1,))])
def test_variance_about_a_huge_mean(shape, axes, G):
    """A mean whose square overflows: folds that meet groups without elements (lanes without rows, chains
    without partial results) must not form the distance to them."""
    rng = np.random.default_rng(shape[0])
    x = (1e20 + 3e16 * rng.standard_normal(shape)).astype(np.float32)
    n = int(np.prod([shape[d] for d in axes]))
    print(f"[case] moments {shape} over {axes} around 1e20", flush=True)
    _expr, got = run_spec(G, _moments_spec(len(shape), axes, n, "f32", False), [x])
    # Deviations are taken from a running mean, a float32 number near 1e20, and rounded with it: off
    # by up to a few of its spacings (8.8e12), four against a deviation of 3e16 change a squared
    # deviation by 2 * 4 * 8.8e12 / 3e16 = 2.3e-3 at worst.
    G.h.compare("var", got[1], x.astype(np.float64).var(axes, keepdims=True).astype(np.float32), 2.5e-3, 0)


@pytest.mark.parametrize("storage", ["f32", "f16"])
@pytest.mark.parametrize("shape", [(300, 64), (1000, 64), (257, 20), (1024, 256), (129, 2000)])
def test_arg_max_down_columns_of_one_workgroup(shape, storage, oracle, G):
    """Eight wavefronts that meet pairwise: ties between them, rows that leave some without a row, NaN."""
    dt = np.float16 if storage == "f16" else np.float32
    rng = np.random.default_rng(shape[0])
    x = rng.integers(-3, 4, shape).astype(dt)                   # many equal maxima: the first one counts
    x[shape[0] // 2, 3] = np.nan
    s = GraphSpec(2)
    v = s.input(storage, (False, False))
    s.output(s.reduce("argmax", v, (0,)), "i32")
    s.output(s.reduce("sum", s.apply("abs", v), (0,)), "f32")
    print(f"[case] arg-max {storage} {shape}", flush=True)
    expr, got = run_spec(G, s, [x])
    assert expr.info()["kernel_class"] == "col" and expr.info()["block_threads"] == 512 and "ewf_finish(" not in expr.source(), expr.info()
    want = oracle.evaluate(s, [x], nthreads=4)
    np.testing.assert_array_equal(got[0], want[0])
    np.testing.assert_array_equal(got[1], want[1])              # small whole numbers: exact
