"""GPU parity of element-wise kernels that stage a permuted operand through LDS, where the tile, its
runs or its rows do not come out even: rows cut inside a vector, runs shorter than or no multiple of
the staging pieces, shares of the staged dimension, few tiles, and tiles dealt to the dies in chunks."""
import numpy as np
import pytest

from tests.test_gpu_ops_and_layouts import G, run_spec  # noqa: F401  (G is the fixture)
from workloads import GraphSpec, configs as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("reading", ["A", "B"])
@pytest.mark.parametrize("n,c,h,w", [(5, 20, 35, 35), (3, 97, 9, 35), (1, 34, 77, 36), (1, 40, 39, 82), (8, 65, 14, 14), (2, 300, 25, 7),
                                     (1, 33, 23, 112), (2, 16, 65, 65), (1, 20, 97, 47), (7, 32, 112, 111), (9, 256, 56, 56)])
def test_stress_expression_on_uneven_planes(n, c, h, w, reading, oracle, G):
    wk = wl.c5_stress(n=n, c=c, h=h, w=w, reading=reading)
    print(f"[case] stress {reading} {n} x {c} x {h} x {w}", flush=True)
    expr, _stats = G.h.check_workload(wk, oracle, nthreads=8)
    info = expr.info()
    assert info["kernel_class"] == "tile" and info["staged_operands"] == ((c if reading == "A" else h) >= 16), info
    assert info["lds_bytes"] <= 80 * 1024, info


@pytest.mark.parametrize("storage", ["f32", "f16"])
@pytest.mark.parametrize("shape", [(1000, 1003), (300, 5000), (513, 700), (16, 70001), (64, 33, 1001), (3, 517, 260)])
def test_sum_with_a_transposed_operand(shape, storage, oracle, G):
    dt = np.float16 if storage == "f16" else np.float32
    rng = np.random.default_rng(shape[-1])
    a = rng.standard_normal(shape).astype(dt)
    # a transposed view that starts inside a wider buffer, so that no run is aligned
    wide = rng.standard_normal(shape[:-2] + (shape[-1], shape[-2] + 3)).astype(dt)
    b = wide[..., 1:1 + shape[-2]].swapaxes(-1, -2)
    nd = len(shape)
    s = GraphSpec(nd)
    x, y, row = s.input(storage, (False,) * nd), s.input(storage, (False,) * nd), s.input("f32", (True,) * (nd - 1) + (False,))
    s.output(s.add(s.mul(x, row), y), "f32")
    r = rng.standard_normal((1,) * (nd - 1) + (shape[-1],)).astype(np.float32)
    print(f"[case] x * row + transposed {storage} {shape}", flush=True)
    expr, got = run_spec(G, s, [a, b, r])
    assert expr.info()["staged_operands"] == 1, expr.info()
    want = oracle.evaluate(s, [a, b, r], nthreads=4)
    # one product and one sum of either sign: relative to the magnitudes of the two terms
    G.h.compare("sum", got[0], want[0], *G.h.ELEMENTWISE, scale=np.abs(a.astype(np.float64) * r) + np.abs(b.astype(np.float64)))


@pytest.mark.parametrize("storage,shape,order,copies", [("f16", (1001, 1003), (1, 0), 3), ("f16", (1001, 1003), (1, 0), 4), ("f32", (640, 512), (1, 0), 3), ("f32", (300, 301), (1, 0), 7),
                                                        ("f16", (25, 300, 16, 3), (1, 0, 3, 2), 2), ("f16", (51, 288, 7), (0, 2, 1), 4), ("f16", (4, 59, 82, 113), (0, 3, 1, 2), 5)])
def test_several_permuted_operands_share_a_tile(storage, shape, order, copies, oracle, G):
    dt = np.float16 if storage == "f16" else np.float32
    rng = np.random.default_rng(copies)
    back = [order.index(d) for d in range(len(shape))]
    xs = [rng.standard_normal(shape).astype(dt)] + [rng.standard_normal([shape[d] for d in order]).astype(dt).transpose(back) for _ in range(copies)]
    s = GraphSpec(len(shape))
    v = s.input(storage, (False,) * len(shape))
    for k in range(copies):
        v = s.add(v, s.mul(s.input(storage, (False,) * len(shape)), s.const(0.5 ** k)))
    s.output(v, "f32")
    print(f"[case] {copies} permuted operands {storage} {shape}", flush=True)
    expr, got = run_spec(G, s, xs)
    assert expr.info()["staged_operands"] == copies and expr.info()["lds_bytes"] <= 160 * 1024, expr.info()
    want = oracle.evaluate(s, xs, nthreads=4)
    # sums of either sign: relative to the magnitudes of the terms
    scale = np.abs(xs[0].astype(np.float64)) + sum(0.5 ** k * np.abs(x.astype(np.float64)) for k, x in enumerate(xs[1:]))
    G.h.compare("sum", got[0], want[0], *G.h.ELEMENTWISE, scale=scale)
