"""GPU parity of rows of which a part waits in LDS: the lengths where that starts, changes and ends, rows whose
last vector is cut, two operands, rows of NaN and infinities next to others, and one that is written over its input."""
import numpy as np
import pytest

from tests.test_gpu_ops_and_layouts import G, run_spec  # noqa: F401  (G is the fixture)
from workloads import GraphSpec

pytestmark = pytest.mark.gpu


def _softmax(storage):
    s = GraphSpec(2)
    x = s.input(storage, (False, False))
    e = s.apply("exp", s.sub(x, s.reduce("max", x, (1,), keep=True)))
    s.output(s.div(e, s.reduce("sum", e, (1,), keep=True)), storage)
    return s


def _lds(G, expr, nbytes):
    info = expr.info()
    assert info["kernel_class"] == "row" and info["block_threads"] == 1024 and info["lds_bytes"] == nbytes, info
    assert ("ewf_ld_lds<" in expr.source()) == (nbytes > 0)


# steps of the row in LDS: none up to 44 registers a thread, then one for each step more, at most four;
# 57344 float32 (56 registers) is the longest row of few rows, 65536 (64) the longest of many
@pytest.mark.parametrize("storage,rows,cols,steps", [("f32", 3 * 64, 45056, 0), ("f32", 3 * 64, 45057, 1), ("f32", 3 * 64, 49154, 2), ("f32", 3 * 64, 57344, 3),
                                                     ("f32", 512, 61441, 4), ("f32", 512, 65536, 4), ("f16", 3 * 64, 90115, 1), ("f16", 3 * 64, 114687, 3)])
def test_rows_partly_in_lds(storage, rows, cols, steps, oracle, G):
    dt = np.float16 if storage == "f16" else np.float32
    rng = np.random.default_rng(cols)
    x = (rng.standard_normal((rows, cols), dtype=np.float32) * 2).astype(dt)
    x[1::8] = np.nan
    x[2::8, cols - 1] = -np.inf
    x[3::8, 0] = np.inf
    spec = _softmax(storage)
    print(f"[case] softmax {storage} {rows} x {cols}", flush=True)
    expr, got = run_spec(G, spec, [x])
    _lds(G, expr, steps * 16384)
    pick = list(range(16)) + [rows - 1]                          # the oracle on rows of every kind
    want = oracle.evaluate(spec, [np.ascontiguousarray(x[pick])], nthreads=8)
    G.h.compare("probabilities", got[0][pick], want[0], *(G.h.HALF if storage == "f16" else G.h.REDUCTION))
    np.testing.assert_array_equal(got[0][16::8].argmax(1), x[16::8].argmax(1))
    torch = G.torch
    xd = torch.from_numpy(x).cuda()
    e2 = G.ewf.Expression(spec)
    ws = G.h.make_workspace(e2, [xd], [xd])
    e2.run([xd], [xd], (), ws, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(xd.cpu().numpy(), got[0])


def test_two_operands_partly_in_lds(oracle, G):
    rows, cols = 130, 27000                                      # 28 registers each, two steps of either in LDS
    rng = np.random.default_rng(7)
    x = rng.standard_normal((rows, cols), dtype=np.float32)
    y = rng.uniform(0.5, 1.5, (rows, cols)).astype(np.float32)
    s = GraphSpec(2)
    a, b = s.input("f32", (False, False)), s.input("f32", (False, False))
    v = s.mul(s.apply("abs", a), b)
    total = s.reduce("sum", v, (1,), keep=True)
    top = s.reduce("max", b, (1,), keep=True)
    s.output(s.add(s.mul(v, s.apply("recip", total)), s.mul(a, top)), "f32")
    s.output(total, "f32")
    print(f"[case] two operands {rows} x {cols}", flush=True)
    expr, got = run_spec(G, s, [x, y])
    _lds(G, expr, 2 * 2 * 16384)
    want = oracle.evaluate(s, [x, y], nthreads=8)
    G.h.compare("out", got[0], want[0], *G.h.REDUCTION)
    G.h.compare("total", got[1], want[1], *G.h.REDUCTION)        # magnitudes: terms of one sign


# rows that are only read: up to 44 registers where there are 512 of them, up to 60 where there are 1024
@pytest.mark.parametrize("rows,vocab,steps", [(512, 24577, 0), (512, 45056, 0), (1024, 49153, 2)])
def test_rows_that_are_only_read(rows, vocab, steps, oracle, G):
    from workloads import configs as wl
    w = wl.c3_softmax_xent(rows=rows, vocab=vocab)
    print(f"[case] {w.name} {rows} x {vocab}", flush=True)
    expr, _stats = G.h.check_workload(w, oracle, nthreads=8)
    _lds(G, expr, steps * 16384)
