"""GPU parity of per-channel sums over planes that are no whole number of vectors: strips of whole channels of an
image's row.  Strips whose last vector is cut, one launch and two, all channels in one strip, operands that vary along
the channels, the plane or both, images with gaps between them, results written over the input."""
import numpy as np
import pytest

from tests.test_gpu_ops_and_layouts import G, run_spec  # noqa: F401  (G is the fixture)
from workloads import GraphSpec

pytestmark = pytest.mark.gpu


def _spec(storage, held):
    s = GraphSpec(4)
    x = s.input(storage, (False,) * 4)
    y = s.input(storage, (False,) * 4)
    h = s.input(storage, held)
    z = s.mul(s.apply("max", s.add(x, h), s.const(0.0)), y)
    s.output(z, storage)
    s.output(s.reduce("sum", s.apply("abs", z), (0, 2, 3)), "f32")
    s.output(s.reduce("max", z, (0, 2, 3), keep=True), "f32")
    s.output(s.apply("sqrt", s.reduce("sum", s.apply("sqr", x), (0, 2, 3))), "f32")
    return s


CHANNEL, PLANE, BOTH = (True, False, True, True), (True, True, False, False), (True, False, False, False)


# [2, 2, 3, 3]: the smallest; [5, 3, 7, 7]: all channels in one strip, its last vector cut; [9, 37, 7, 7] and [3, 70, 15, 15]: a last strip
# with fewer channels and a cut vector; [40, 150, 9, 9], [33, 40, 31, 31]: workgroups share the images, partials folded by a thread a
# channel; [400, 33, 7, 7] by lanes; [20, 30, 33, 33]: vectors cut in every strip; [6, 50, 5, 6]: two elements over
SHAPES = [((2, 2, 3, 3), CHANNEL), ((5, 3, 7, 7), PLANE), ((9, 37, 7, 7), CHANNEL), ((3, 70, 15, 15), BOTH), ((40, 150, 9, 9), CHANNEL),
          ((33, 40, 31, 31), CHANNEL), ((400, 33, 7, 7), BOTH), ((20, 30, 33, 33), PLANE), ((6, 50, 5, 6), CHANNEL)]


# (float16 planes of more than 600 bytes are rows of their own)
@pytest.mark.parametrize("shape,held,storage", [s + ("f32",) for s in SHAPES] + [s + ("f16",) for s in SHAPES if s[0][2] * s[0][3] <= 300])
def test_sums_over_ragged_planes(shape, held, storage, oracle, G):
    dt = np.float32 if storage == "f32" else np.float16
    n, c, hh, ww = shape
    rng = np.random.default_rng(n * c + hh)
    buf = rng.standard_normal((n, c + 2, hh, ww)).astype(dt)
    x = buf[:, 1:1 + c]                                          # images with a gap between them
    if c > 2: buf[0, 2, 0, 1] = np.nan                           # channel 1 only
    y = rng.uniform(-1, 1, shape).astype(dt)
    h = rng.standard_normal([1 if b else e for b, e in zip(held, shape)]).astype(dt)
    spec = _spec(storage, held)
    print(f"[case] {storage} {shape} {held}", flush=True)
    expr, got = run_spec(G, spec, [x, y, h])
    assert expr.info()["kernel_class"] == "col" and "sm_flat" in expr.source(), expr.info()
    want = oracle.evaluate(spec, [x, y, h], nthreads=4)
    G.h.compare("z", got[0], want[0], *(G.h.ELEMENTWISE if storage == "f32" else G.h.HALF))
    G.h.compare("sum", got[1], want[1], *G.h.REDUCTION)          # magnitudes and squares: terms of one sign
    G.h.compare("max", got[2], want[2], *G.h.ELEMENTWISE)        # one element, as exact as z before it is stored
    G.h.compare("norm", got[3], want[3], *G.h.REDUCTION)
    # over the second operand, in place
    torch = G.torch
    bd, yd, hd = (torch.from_numpy(a).cuda() for a in (buf, y, h))
    xd = bd[:, 1:1 + c]
    e2 = G.ewf.Expression(spec)
    outs = [yd] + G.h.alloc_outputs(e2, spec, [xd, yd, hd])[1:]
    ws = G.h.make_workspace(e2, [xd, yd, hd], outs)
    e2.run([xd, yd, hd], outs, (), ws, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    for a, b in zip(outs, got):
        np.testing.assert_array_equal(a.cpu().numpy(), b)
