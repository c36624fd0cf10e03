"""The marks of a batch (new out-edges of each source, which propagation leaves out) are gone when it ends: the nodes that got an
edge change their features afterwards, and a mark left over would keep that from one of their neighbours.  Numbers of sources
around the one from which the marks have a launch of their own."""
import numpy as np
import pytest

import synth
from util import Harness
from test_gpu_edge_cases import tiny_model, INS

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("agg,sources", [("max", 1), ("max", 513), ("sum", 4095), ("max", 4096), ("max", 4097), ("sum", 9000), ("max", 20000)])
def test_marks_are_cleared(agg, sources):
    n = 30000
    rng = np.random.default_rng(sources)
    src, dst = synth.keys_to_edges(np.unique(synth.edge_keys(rng.integers(0, n, 3 * n).astype(np.int32), rng.integers(0, n, 3 * n).astype(np.int32))))
    src, dst = src[src != dst], dst[src != dst]
    exact = agg == "max"
    h = Harness(graph=(n, src, dst), X=rng.standard_normal((n, 4)).astype(np.float32), model=tiny_model("sage", agg, (4, 3), seed=1),
                precision="f32" if exact else "f64", dense_threshold=-1)
    who = rng.choice(n, size=sources, replace=False).astype(np.int32)
    for k in range(2):
        h.step(np.full(sources, INS, np.uint8), who, ((who + 11 + k) % n).astype(np.int32), exact=exact)
        h.feature_step(who, rng.standard_normal((sources, 4)).astype(np.float32), exact=exact)
    h.check_state(exact=exact)
    h.ink.close()
