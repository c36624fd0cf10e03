"""The rows to transform in one launch: graphs of one tile of the bitmap (16384 nodes) and one node more, changed sources and nodes of
changed degree up to what the launch marks itself and beyond."""
import numpy as np
import pytest

from util import Harness
from test_gpu_edge_cases import tiny_model, INS, DEL
from test_gpu_layer_one import ring_with_hub

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,agg,exact", [("sage", "max", True), ("sage", "mean", False), ("gcn", "gcn_sym", False)])
@pytest.mark.parametrize("n", [64, 130, 16383, 16384, 16385])
def test_one_tile_of_nodes(n, kind, agg, exact):
    src, dst = ring_with_hub(n, min(60, n - 2), n)
    rng = np.random.default_rng(n)
    dims = (7, 6, 5)
    X = rng.integers(-3, 4, size=(n, dims[0])).astype(np.float32)
    h = Harness(graph=(n, src, dst), X=X, model=tiny_model(kind, agg, dims, seed=3), precision="f32" if exact else "f64", slack=0.1)
    for size in (40, 300):
        s, d = rng.integers(0, n, size=size).astype(np.int32), rng.integers(0, n, size=size).astype(np.int32)
        s[0] = d[1] = n - 1
        h.step(np.full(size, INS, np.uint8), s, d, exact=exact, tol=1e-5)
        h.step(np.full(size, DEL, np.uint8), s, d, exact=exact, tol=1e-5)
    for size in (1, min(n, 4000), min(n, 4200)):
        ids = rng.choice(n, size=size, replace=False).astype(np.int32)
        h.feature_step(ids, rng.integers(-3, 4, size=(size, dims[0])).astype(np.float32), exact=exact, tol=1e-5)
    h.check_state(exact=exact, tol=1e-5); h.check_graph()
    h.ink.close()
