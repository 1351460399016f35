"""GPU parity of sums down columns whose number or alignment allows narrow accesses only and that are read in wide
vectors all the same: the last vector cut, a last strip narrower than a vector, rows at odd elements, one launch and two."""
import numpy as np
import pytest

from tests.test_gpu_ops_and_layouts import G, run_spec  # noqa: F401  (G is the fixture)
from workloads import GraphSpec

pytestmark = pytest.mark.gpu


def _spec(storage, ndim, axis):
    s = GraphSpec(ndim)
    x = s.input(storage, (False,) * ndim)
    k = s.input("f32", tuple(d == axis for d in range(ndim)))      # one value per column
    d = s.sub(x, k)
    s.output(s.reduce("sum", s.apply("sqr", d), (axis,)), "f32")
    s.output(s.reduce("max", d, (axis,)), "f32")
    s.output(s.reduce("argmax", x, (axis,)), "i32")
    return s


# [40960, 255]: one strip of 64 lanes, its last vector cut; [12288, 769]: a last strip of one column; [45056, 256]: whole
# vectors that start at odd elements; [24, 200, 2001]: tiles over an outer index; [64, 90, 509]: whole columns in one launch
SHAPES = [((40960, 255), 0, "f32"), ((12288, 769), 0, "f32"), ((45056, 256), 0, "f32"), ((24, 200, 2001), 1, "f32"),
          ((90000, 509), 0, "f16"), ((64, 1000, 999), 1, "f16"), ((64, 90, 509), 1, "f16"), ((128, 64, 253), 1, "f32")]


@pytest.mark.parametrize("shape,axis,storage", SHAPES)
def test_columns_in_vectors_of_any_alignment(shape, axis, storage, oracle, G):
    dt = np.float32 if storage == "f32" else np.float16
    rng = np.random.default_rng(sum(shape))
    buf = rng.standard_normal(shape[:-1] + (shape[-1] + 3,)).astype(dt)
    x = buf[..., 1:1 + shape[-1]]                                  # rows from an odd element, gaps between them
    x[(3,) * (x.ndim - 1) + (shape[-1] - 1,)] = np.nan             # the last column only
    x[(5,) * (x.ndim - 1) + (0,)] = -np.inf
    k = rng.standard_normal([1 if d == axis else e for d, e in enumerate(shape)]).astype(np.float32)
    spec = _spec(storage, len(shape), axis)
    print(f"[case] {storage} {shape} {axis}", flush=True)
    expr, got = run_spec(G, spec, [x, k])
    assert expr.info()["kernel_class"] == "col" and "ewf_ld_u<" in expr.source().split("ewf_kernel")[1], expr.info()
    want = oracle.evaluate(spec, [x, k], nthreads=4)
    G.h.compare("sum", got[0], want[0], *G.h.REDUCTION)            # terms of one sign
    G.h.compare("max", got[1], want[1], *G.h.ELEMENTWISE)          # one element's difference
    np.testing.assert_array_equal(got[2], want[2])
