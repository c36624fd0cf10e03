"""The transform of few rows (tiles of 16 rows and 16 columns) and of many: every count around a tile and around the line
between the two, widths with remainders on both sides, every kind of layer."""
import numpy as np
import pytest

import synth
from util import Harness
from test_gpu_edge_cases import tiny_model, INS, DEL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,agg,dims", [("sage", "max", (3, 1, 5)), ("sage", "min", (33, 130, 16)), ("sage", "max", (128, 128, 128)),
                                           ("sage", "max", (200, 256, 47)), ("sage", "mean", (50, 121, 7)), ("gin", "sum", (40, 17, 172)),
                                           ("gin", "max", (64, 200, 9)), ("gcn", "gcn_sym", (70, 256, 41)), ("gcn", "gcn_sym", (16, 33, 200))])
@pytest.mark.parametrize("n", [1, 15, 17, 2047, 2049])
def test_row_counts(kind, agg, dims, n):
    rng = np.random.default_rng(n + dims[0])
    src, dst = rng.integers(0, n, 4 * n), rng.integers(0, n, 4 * n)
    keys = np.unique(synth.edge_keys(src.astype(np.int32), dst.astype(np.int32))[src != dst])
    src, dst = synth.keys_to_edges(keys)
    exact = agg in ("max", "min")
    X = rng.standard_normal((n, dims[0])).astype(np.float32)
    h = Harness(graph=(n, src, dst), X=X, model=tiny_model(kind, agg, dims, seed=n, hidden=24), precision="f32" if exact else "f64")
    h.check_state(exact=exact)
    for k in (1, 7, 300):
        k = min(k, src.size)
        if k == 0:
            continue
        pick = rng.choice(h.keys.size, size=k, replace=False)
        s, d = synth.keys_to_edges(h.keys[pick])
        h.step(np.full(k, DEL, np.uint8), s.astype(np.int32), d.astype(np.int32), exact=exact)
        h.step(np.full(k, INS, np.uint8), s.astype(np.int32), d.astype(np.int32), exact=exact)
        h.check_state(exact=exact)
    h.ink.close()
