"""The changed rows of a layer, their order and the events they propagate, at row counts around a workgroup (256 rows),
around the forms of the emission (one workgroup up to 4096 rows, one row a thread up to 262144, eight beyond) and with
rows that did not change among them."""
import numpy as np
import pytest

import synth
from util import Harness
from test_gpu_edge_cases import tiny_model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_rows", [4096, 4097, 4351, 4352, 4353, 262143, 262144, 262145, 264193])
@pytest.mark.parametrize("agg", ["max", "sum"])
def test_changed_rows(n_rows, agg):
    n = n_rows + 1000
    rng = np.random.default_rng(n_rows)
    # every third of the listed nodes keeps its row; the others reach one to three nodes each
    keys = np.unique(synth.edge_keys(rng.integers(0, n, size=2 * n).astype(np.int32), rng.integers(0, n, size=2 * n).astype(np.int32)))
    src, dst = synth.keys_to_edges(keys)
    off = src != dst
    X = rng.integers(-3, 4, size=(n, 4)).astype(np.float32)
    exact = agg == "max"
    h = Harness(graph=(n, src[off], dst[off]), X=X, model=tiny_model("sage" if exact else "gin", agg, (4, 8, 5), seed=3, hidden=8),
                dense_threshold=-1, precision="f32" if exact else "f64")
    ids = np.sort(rng.choice(n, size=n_rows, replace=False)).astype(np.int32)
    rows = X[ids] + 1
    rows[::3] = X[ids[::3]]
    h.feature_step(ids, rows, exact=exact)
    changed = np.delete(ids, np.s_[::3])
    L = h.ink.stats()["layers"][0]
    assert (L["n_sources"], L["n_events"]) == (len(changed), int(np.isin(src[off], changed).sum()))
    h.check_state(exact=exact)
    h.ink.close()
