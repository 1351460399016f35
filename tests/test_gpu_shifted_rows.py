"""GPU parity of long rows whose vectors start on the output's cache lines: every remainder of a row's length, rows
aligned to a vector but not to a line, a float32 result of float16 rows, input and output of different pitches, rows of
NaN next to others, a result written over the input, workgroups that take several rows in turn."""
import numpy as np
import pytest

from tests.test_gpu_ops_and_layouts import G  # noqa: F401  (the fixture)
from workloads import GraphSpec

pytestmark = pytest.mark.gpu


def _spec(storage, out):
    s = GraphSpec(2)
    x = s.input(storage, (False, False))
    e = s.apply("exp", s.sub(x, s.reduce("max", x, (1,), keep=True)))
    total = s.reduce("sum", e, (1,), keep=True)
    s.output(s.div(e, total), out)
    s.output(total, "f32")
    return s


CASES = [("f32", "f32", 2600, c, 0) for c in (5001, 5002, 5003)] + [("f32", "f32", 4200, 5004, 0)] + [("f16", "f16", 5100, c, 0) for c in range(5001, 5008)]
CASES += [("f32", "f32", 2600, 5003, 7), ("f16", "f16", 5100, 5003, 5), ("f16", "f32", 3400, 5005, 0), ("f32", "f32", 1024, 12301, 0), ("f32", "f32", 800, 16383, 0), ("f32", "f32", 600, 24577, 1)]


@pytest.mark.parametrize("storage,out,rows,cols,gap", CASES)
def test_rows_that_start_inside_a_line(storage, out, rows, cols, gap, oracle, G):
    _check(storage, out, rows, cols, gap, oracle, G)


# more than 8192 rows, or a grid of fewer workgroups than rows: a workgroup's rows start at different distances from a line
@pytest.mark.parametrize("storage,rows,cols,opts", [("f16", 10000, 5003, {}), ("f32", 8193, 5001, {}), ("f32", 2600, 5003, {"max_blocks": 301}), ("f16", 5100, 5005, {"max_blocks": 64})])
def test_rows_in_turn(storage, rows, cols, opts, oracle, G):
    _check(storage, storage, rows, cols, 0, oracle, G, **opts)


def _check(storage, out, rows, cols, gap, oracle, G, **opts):
    torch = G.torch
    dt = np.float16 if storage == "f16" else np.float32
    rng = np.random.default_rng(cols + gap)
    buf = (rng.standard_normal((rows, cols + gap), dtype=np.float32) * 2).astype(dt)
    x = buf[:, gap // 2:gap // 2 + cols]
    x[5::64] = np.nan
    x[6::64, -1] = -np.inf
    x[7::64, 0] = 1e4                                            # the probabilities' only one, at either end
    x[8::64, -1] = 1e4
    spec = _spec(storage, out)
    print(f"[case] {storage} to {out} {rows} x {cols} pitch {cols + gap}", flush=True)
    xd = torch.from_numpy(buf).cuda()[:, gap // 2:gap // 2 + cols]
    expr = G.ewf.Expression(spec, **opts)
    outs = G.h.alloc_outputs(expr, spec, [xd])
    guard = torch.full((rows * cols + 64,), 7.0, dtype=outs[0].dtype, device="cuda")        # what lies behind the last row stays
    outs[0] = guard[:rows * cols].view(rows, cols)
    ws = G.h.make_workspace(expr, [xd], outs)
    stream = torch.cuda.current_stream().cuda_stream
    expr.run([xd], outs, (), ws, stream)
    torch.cuda.synchronize()
    assert expr.info()["kernel_class"] == "row" and "head_" in expr.source(), expr.info()
    assert ("row += gridDim.x" in expr.source()) == (rows > 8192 or "max_blocks" in opts)
    assert (guard[rows * cols:] == 7.0).all()
    pick = list(range(70)) + [rows - 2, rows - 1]                # every distance of a row's start from a line
    want = oracle.evaluate(spec, [np.ascontiguousarray(x[pick])], nthreads=8)
    got = [o.cpu().numpy() for o in outs]
    G.h.compare("probabilities", got[0][pick], want[0], *(G.h.HALF if out == "f16" else G.h.REDUCTION))
    G.h.compare("total", got[1][pick], want[1], *G.h.REDUCTION)
    if storage == out:                                           # over the input
        outs2 = [xd, outs[1]]
        e2 = G.ewf.Expression(spec, **opts)
        e2.run([xd], outs2, (), G.h.make_workspace(e2, [xd], outs2), stream)
        torch.cuda.synchronize()
        if gap == 0: np.testing.assert_array_equal(xd.cpu().numpy(), got[0])
        else: G.h.compare("in place", xd.cpu().numpy()[pick], want[0], *(G.h.HALF if out == "f16" else G.h.REDUCTION))
