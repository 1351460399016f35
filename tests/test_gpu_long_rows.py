"""GPU parity of softmax cross-entropy and its gradient at the row lengths where the plan changes between
rows held in registers, up to 56 of them per thread, and rows split over workgroups."""
import pytest

from tests.test_gpu_ops_and_layouts import G  # noqa: F401  (the fixture)
from workloads import configs as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("vocab,forward,backward", [(24576, "row", "row"), (24577, "tile_reduce", "row"), (32769, "tile_reduce", "row"), (49153, "tile_reduce", "row"),
                                                    (50257, "tile_reduce", "row"), (57344, "tile_reduce", "row"), (57345, "tile_reduce", "multi")])
def test_softmax_cross_entropy_where_the_plan_changes(vocab, forward, backward, oracle, G):
    for make, kind in ((wl.c3_softmax_xent, forward), (wl.c3_softmax_xent_backward, backward)):
        w = make(rows=131, vocab=vocab)
        print(f"[case] {w.name} 131 x {vocab}", flush=True)
        expr, _stats = G.h.check_workload(w, oracle, nthreads=8)
        assert expr.info()["kernel_class"] in (kind, "multi" if kind == "tile_reduce" else kind), expr.info()
