"""Where the default dense_threshold lies: the fraction of the edges on either side of which a layer groups its
events or re-aggregates every node, by aggregator, width, event count, and for large graphs by node."""
import numpy as np
import pytest

import synth
from util import Harness
from test_gpu_edge_cases import tiny_model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("agg,d,n,sources,dense", [
    ("max", 64, 4000, 1400, 0), ("max", 64, 4000, 1401, 1), ("min", 65, 4000, 1800, 0), ("min", 65, 4000, 1801, 1),
    ("max", 20, 1200, 819, 0), ("max", 20, 1200, 820, 1), ("sum", 64, 4000, 2999, 0), ("mean", 20, 4000, 3001, 1)])
def test_default_threshold(agg, d, n, sources, dense):
    rng = np.random.default_rng(n + sources)
    v = np.arange(n)
    src = np.repeat(v, 5)                                   # 5 out-edges each: 5 events per changed row
    dst = (src + 1 + 7 * np.tile(np.arange(5), n)) % n
    src, dst = synth.keys_to_edges(np.unique(synth.edge_keys(src.astype(np.int32), dst.astype(np.int32))))
    exact = agg in ("max", "min")
    X = rng.integers(-3, 4, size=(n, d)).astype(np.float32)
    h = Harness(graph=(n, src, dst), X=X, model=tiny_model("sage", agg, (d, 12, 6), seed=d), precision="f32" if exact else "f64")
    ids = np.sort(rng.choice(n, size=sources, replace=False)).astype(np.int32)
    h.feature_step(ids, X[ids] + 1, exact=exact)
    L = h.ink.stats()["layers"][0]
    assert L["n_events"] == 5 * sources and L["dense"] == dense
    h.check_state(exact=exact)
    h.ink.close()


@pytest.mark.parametrize("n,fan,d,sources,dense", [
    (300_000, 2, 4, 105_000, 0), (300_000, 2, 4, 105_001, 1),     # the nodes do not count yet: .35
    (700_000, 5, 4, 445_000, 0), (700_000, 5, 4, 445_001, 1),     # .35 of 3.5 M edges + 2.5 x 400 000 nodes
    (400_000, 4, 68, 180_000, 0), (400_000, 4, 68, 180_001, 1),   # wide rows, no edge update: .45
    (1_200_000, 3, 4, 900_000, 0), (1_200_000, 3, 4, 900_001, 1)])   # at most .75
def test_default_threshold_of_large_graphs(n, fan, d, sources, dense):
    v = np.arange(n)
    dst = (np.repeat(v, fan) + 1 + 7 * np.tile(np.arange(fan), n)) % n
    src, dst = synth.keys_to_edges(np.unique(synth.edge_keys(np.repeat(v, fan).astype(np.int32), dst.astype(np.int32))))
    rng = np.random.default_rng(n)
    X = rng.integers(-3, 4, size=(n, d)).astype(np.float32)
    h = Harness(graph=(n, src, dst), X=X, model=tiny_model("sage", "max", (d, 3), seed=d), precision="f32")
    ids = np.sort(rng.choice(n, size=sources, replace=False)).astype(np.int32)
    h.feature_step(ids, X[ids] + 1)
    L = h.ink.stats()["layers"][0]
    assert L["n_events"] == fan * sources and L["dense"] == dense
    h.check_state()
    h.ink.close()


@pytest.mark.parametrize("n,dense", [(300_000, 1), (302_399, 1), (302_401, 0), (400_000, 0)])
def test_default_threshold_of_edge_updates(n, dense):
    """60 000 events on 120 000 edges: .45 of them, and 6000 more from 302 400 nodes on."""
    v = np.arange(60_000, dtype=np.int32)
    X = np.random.default_rng(n).integers(-3, 4, size=(n, 68)).astype(np.float32)
    h = Harness(graph=(n, v, v + 1), X=X, model=tiny_model("sage", "max", (68, 3), seed=5), precision="f32")
    h.step(np.zeros(60_000, np.uint8), v, v + 9)
    L = h.ink.stats()["layers"][0]
    assert L["n_events"] == 60_000 and L["dense"] == dense
    h.check_state()
    h.ink.close()
