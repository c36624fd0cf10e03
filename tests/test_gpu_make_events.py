"""Events of layers too long for one workgroup, by how many sources a wave's share of them has: hubs, a few events a
source, more sources than are brought into LDS, sources without out-edges between the others."""
import numpy as np
import pytest

import synth
from util import Harness
from test_gpu_edge_cases import tiny_model, INS, DEL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,agg", [("sage", "max"), ("gin", "sum")])
@pytest.mark.parametrize("degrees", [[1], [0, 1], [0, 0, 0, 0, 0, 1], [3], [2, 3, 4], [20], [0, 40, 1], [900, 0, 1, 2]])
def test_sources_of_a_wave(kind, agg, degrees):
    n_src = -(-6000 // sum(degrees)) * len(degrees) if sum(degrees) < 100 else 80 * len(degrees)     # 6000 events, or 72000 of hubs
    rng = np.random.default_rng(sum(degrees) + n_src)
    n = n_src + 3000
    k = np.resize(degrees, n_src)
    src = np.repeat(np.arange(n_src), k)
    dst = np.concatenate([rng.choice(3000, size=c, replace=False) for c in k]) + n_src
    src, dst = synth.keys_to_edges(np.unique(synth.edge_keys(src.astype(np.int32), dst.astype(np.int32))))
    assert src.size > 4096
    exact = agg == "max"
    X = rng.integers(-3, 4, size=(n, 6)).astype(np.float32)
    h = Harness(graph=(n, src, dst), X=X, model=tiny_model(kind, agg, (6, 5, 4), seed=1, hidden=8), dense_threshold=-1,
                precision="f32" if exact else "f64")
    new = rng.integers(-3, 4, size=(n_src, 6)).astype(np.float32) + np.float32(0.5)
    h.feature_step(np.arange(n_src, dtype=np.int32), new, exact=exact)
    h.check_state(exact=exact)
    gone = rng.choice(src.size, size=300, replace=False)               # removed and inserted edges on both sides of the others
    op = np.r_[np.full(300, DEL), np.full(9, INS)].astype(np.uint8)
    h.step(op, np.r_[src[gone], np.full(9, n - 1)].astype(np.int32), np.r_[dst[gone], np.arange(9)].astype(np.int32), exact=exact)
    h.check_state(exact=exact)
    h.ink.close()
