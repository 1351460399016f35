"""GPU parity of element-wise kernels whose tiles are as many whole rows as make up whole cache lines: the last tile
cut, one value a column and one a row beside the tensor, rows with gaps between them, results over the input."""
import numpy as np
import pytest

from tests.test_gpu_ops_and_layouts import G, run_spec  # noqa: F401  (G is the fixture)
from workloads import GraphSpec

pytestmark = pytest.mark.gpu


def _spec(storage):
    s = GraphSpec(2)
    x = s.input(storage, (False, False))
    m = s.input("f32", (True, False))
    r = s.input("f32", (False, True))
    s.output(s.mul(s.sub(x, m), r), storage)
    return s


# (shape, rows of a tile): half lines, quarters, 4 bytes off; float16 of 15.625 lines
@pytest.mark.parametrize("rows,cols,storage,tile_rows", [(20001, 816, "f32", 2), (65537, 1000, "f32", 8), (100001, 67, "f32", 32),
                                                         (140003, 99, "f32", 32), (60005, 1000, "f16", 8), (30011, 1776, "f32", 4)])
def test_tiles_of_whole_lines(rows, cols, storage, tile_rows, oracle, G):
    dt = np.float32 if storage == "f32" else np.float16
    rng = np.random.default_rng(rows + cols)
    x = rng.standard_normal((rows, cols), dtype=np.float32).astype(dt)
    m = rng.standard_normal((1, cols)).astype(np.float32)
    r = rng.uniform(0.5, 2, (rows, 1)).astype(np.float32)
    spec = _spec(storage)
    print(f"[case] {storage} {rows} {cols}", flush=True)
    expr, got = run_spec(G, spec, [x, m, r])
    assert expr.info()["kernel_class"] == "tile" and expr.info()["tile"] == (tile_rows, cols), expr.info()
    want = oracle.evaluate(spec, [x, m, r], nthreads=4)
    tol = G.h.ELEMENTWISE if storage == "f32" else G.h.HALF
    G.h.compare("y", got[0], want[0], *tol)
    torch = G.torch
    xd, md, rd = (torch.from_numpy(a).cuda() for a in (x, m, r))
    e2 = G.ewf.Expression(spec)
    e2.run([xd, md, rd], [xd], (), None, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(xd.cpu().numpy(), got[0])
