"""A reduction's result is the same bits in every thread of a workgroup of 1024: what sixteen wavefronts hold is met in one
order, also where the order shows (zeros of either sign, means with their counts)."""
import numpy as np
import pytest

from tests.test_gpu_ops_and_layouts import G, run_spec  # noqa: F401  (G is the fixture)
from workloads import GraphSpec

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("op", ["min", "max"])
def test_zeros_of_either_sign_across_wavefronts(op, oracle, G):
    rows, cols = 160, 40000
    sign = 1.0 if op == "min" else -1.0
    rng = np.random.default_rng(3)
    x = (rng.uniform(0.5, 1.5, (rows, cols)) * sign).astype(np.float32)
    for r in range(rows):                                        # wavefront w of a row's first 4096 elements: 256 w ...
        w = rng.permutation(16)
        x[r, 256 * w[:1 + r % 15] + 7] = 0.0
        x[r, 256 * w[1 + r % 15:] + 7] = -0.0
    s = GraphSpec(2)
    v = s.input("f32", (False, False))
    m = s.reduce(op, v, (1,), keep=True)
    s.output(s.div(s.add(s.apply("abs", v), s.const(1.0)), m), "f32")       # an infinity of the extreme's sign
    # (NaN-aware rules: the hardware maximum orders the zeros)
    print(f"[case] {op}", flush=True)
    expr, got = run_spec(G, s, [x], plain_extremes=1)
    assert expr.info()["kernel_class"] == "row" and expr.info()["block_threads"] == 1024, expr.info()
    assert np.isinf(got[0]).all()
    signs = np.signbit(got[0])
    assert (signs == signs[:, :1]).all()
