"""Layers whose events go through the device-wide sort, at every digit width and tile size its plan can choose: the
bits of the node ids and the number of events on either side of 2^18 (tile) and 2^20 (digit) decide."""
import numpy as np
import pytest

import synth
from util import Harness
from test_gpu_edge_cases import tiny_model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,fan,sources", [
    (1500, 10, 500),            # 11 bits: one pass of 11
    (40_000, 5, 820),           # 16 bits: two of 8
    (140_000, 5, 52_428),       # 18 bits: two of 9, 262 140 events: short tiles
    (140_000, 5, 52_429),       # 262 145 events: long tiles
    (600_000, 8, 5_000),        # 20 bits: two of 11
    (600_000, 8, 131_072),      # 2^20 events: two of 11
    (600_000, 8, 131_073),      # three of 8: the sorted pair ends in the other buffer
    (140_000, 10, 104_900),     # 18 bits, more than 2^20 events: two of 9
])
@pytest.mark.parametrize("agg", ["max", "sum"])
def test_event_sort(n, fan, sources, agg):
    rng = np.random.default_rng(sources)
    v = np.arange(n)
    src = np.repeat(v, fan)                                  # fan out-edges each: fan events per changed row
    dst = (src + 1 + 131 * np.tile(np.arange(fan), n)) % n
    src, dst = synth.keys_to_edges(np.unique(synth.edge_keys(src.astype(np.int32), dst.astype(np.int32))))
    X = rng.integers(-3, 4, size=(n, 4)).astype(np.float32)
    h = Harness(graph=(n, src, dst), X=X, model=tiny_model("sage", agg, (4, 3), seed=fan), dense_threshold=-1,
                precision="f32" if agg == "max" else "f64")
    ids = np.sort(rng.choice(n, size=sources, replace=False)).astype(np.int32)
    h.feature_step(ids, X[ids] + 1, exact=agg == "max")
    L = h.ink.stats()["layers"][0]
    assert L["n_events"] == fan * sources and not L["dense"]
    h.check_state(exact=agg == "max")
    h.ink.close()
