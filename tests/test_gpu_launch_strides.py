"""More chunks of long rows than a short launch has workgroups: the slices of every chunk are taken by the grid's stride."""
import numpy as np
import pytest

import synth
from util import Harness
from test_gpu_edge_cases import tiny_model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("agg,d", [("max", 256), ("min", 100), ("max", 33)])
def test_chunks_beyond_the_grid(agg, d):
    n, fan = 6000, 150
    rng = np.random.default_rng(d)
    src, dst = synth.keys_to_edges(np.unique(synth.edge_keys(rng.integers(0, n, n * fan).astype(np.int32), rng.integers(0, n, n * fan).astype(np.int32))))
    src, dst = src[src != dst], dst[src != dst]
    h = Harness(graph=(n, src, dst), X=rng.standard_normal((n, d)).astype(np.float32), model=tiny_model("sage", agg, (d, 5), seed=d), dense_threshold=-1)
    ids = rng.choice(n, size=n // 2, replace=False).astype(np.int32)
    h.feature_step(ids, rng.standard_normal((ids.size, d)).astype(np.float32))
    assert h.ink.stats()["layers"][0]["n_regather_nb_long"] > 1024 * fan       # nothing was expected of this layer: the smallest grid
    h.check_state()
    h.ink.close()
