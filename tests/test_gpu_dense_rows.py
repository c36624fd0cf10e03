"""Layers that re-aggregate every node leave rows without in-neighbours alone unless they lost their last edge in the
batch: nodes that lose all, some and none of their edges, that get their first, and that never had one."""
import numpy as np
import pytest

import synth
from util import Harness
from test_gpu_edge_cases import tiny_model, INS, DEL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("agg,d", [("max", 5), ("min", 64), ("max", 128), ("min", 200), ("max", 300)])
@pytest.mark.parametrize("n", [700, 9001])
def test_rows_without_neighbours(agg, d, n):
    rng = np.random.default_rng(d + n)
    lengths = np.zeros(n, np.int64)
    lengths[:60] = np.arange(60) % 4
    lengths[60:63] = [257, 300, 600]
    src = np.concatenate([rng.choice(np.arange(64, n), size=k, replace=False) for k in lengths])
    dst = np.repeat(np.arange(n), lengths)
    src, dst = synth.keys_to_edges(np.unique(synth.edge_keys(src.astype(np.int32), dst.astype(np.int32))))
    X = rng.integers(-2, 3, size=(n, d)).astype(np.float32)
    h = Harness(graph=(n, src, dst), X=X, model=tiny_model("sage", agg, (d, 6, 3), seed=d), dense_threshold=1e-6)
    for gone in (np.isin(dst, [1, 2, 3, 62]), np.isin(dst, [5, 61]) & (np.arange(dst.size) % 2 == 0)):
        op = np.r_[np.full(gone.sum(), DEL), np.full(3, INS)].astype(np.uint8)
        bs = np.r_[src[gone], [n - 1, n - 2, n - 3]].astype(np.int32)
        bd = np.r_[dst[gone], [4, 8, 200]].astype(np.int32)
        h.step(op, bs, bd)
        assert h.ink.stats()["layers"][0]["dense"] and h.ink.stats()["layers"][0]["n_targets"] == n
        h.check_state(); h.check_graph(); h.check_bound(max_nodes=n)
        h.step((1 - op)[::-1].copy(), bs[::-1].copy(), bd[::-1].copy())
        h.check_state(); h.check_bound(max_nodes=n)
    h.ink.close()


@pytest.mark.parametrize("affected", [False, True])
def test_a_dense_layer_passes_on_what_changed(affected):
    """Targets that lose edges without effect are not counted among the nodes whose aggregate changed: an update transforms the
    rows that changed and no others, the baseline propagates from these and the changed edges' sources alone."""
    n, hubs, rng = 4000, 50, np.random.default_rng(1)
    src = np.concatenate([np.r_[3000 + i, rng.choice(np.arange(100, 2900), size=20, replace=False)] for i in range(hubs)])
    dst = np.repeat(np.arange(hubs), 21)
    src, dst = synth.keys_to_edges(np.unique(synth.edge_keys(src.astype(np.int32), dst.astype(np.int32))))
    X = rng.random((n, 8)).astype(np.float32)
    X[3000:3000 + hubs] = 9.0                                # one neighbour of every hub holds all of its dimensions
    h = Harness(graph=(n, src, dst), X=X, model=tiny_model("sage", "max", (8, 6, 3), seed=1), dense_threshold=1e-6)
    low = np.flatnonzero(src < 2900)
    low = low[np.unique(dst[low], return_index=True)[1]]     # one edge of every hub that holds nothing
    top = np.flatnonzero((src >= 3000) & (dst < 7))          # and what holds everything of seven of them
    gone = np.r_[low, top]
    h.step(np.full(gone.size, DEL, np.uint8), src[gone].astype(np.int32), dst[gone].astype(np.int32), affected=affected)
    L = h.ink.stats()["layers"]
    assert L[0]["dense"] and L[0]["n_transformed"] == 7 and L[0]["n_changed"] == 7 and L[1]["n_sources"] == 7
    h.check_state()
    h.ink.close()
