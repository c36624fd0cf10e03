"""Targets whose event segment is reduced by many waves: lengths around the limits (128 in short launches, 64, 128 or 256 in
larger ones), around multiples of a chunk (128 or 256), and a hub with thousands, with every lane width and with events of
all three kinds in one segment."""
import numpy as np
import pytest

import synth
from util import Harness
from test_gpu_edge_cases import tiny_model, INS, DEL

pytestmark = pytest.mark.gpu


def hub_graph(n_src, fan, n, seed):
    """Sources 2 .. n_src + 1 point to hub 0 (and a third of them to hub 1) and to `fan` random other nodes."""
    rng = np.random.default_rng(seed)
    s = np.arange(2, n_src + 2)
    src = [s, s[::3], np.repeat(s, fan)]
    dst = [np.zeros(n_src, np.int64), np.ones(len(s[::3]), np.int64), rng.integers(n_src + 2, n, size=n_src * fan)]
    keys = np.unique(synth.edge_keys(np.concatenate(src).astype(np.int32), np.concatenate(dst).astype(np.int32)))
    return synth.keys_to_edges(keys)


@pytest.mark.parametrize("kind,agg,d", [("sage", "max", 20), ("sage", "min", 100), ("gin", "max", 256), ("sage", "sum", 40),
                                        ("sage", "mean", 128), ("gin", "sum", 300), ("gcn", "gcn_sym", 70)])
@pytest.mark.parametrize("n_src,fan", [(127, 1), (129, 1), (255, 45), (257, 45), (513, 20), (3000, 5)])
def test_hub_segments(kind, agg, d, n_src, fan):
    n = n_src + 9000
    dims = (d, d if kind == "gcn" else 24, 6)
    src, dst = hub_graph(n_src, fan, n, n_src + d)
    rng = np.random.default_rng(n_src)
    exact = agg in ("max", "min")
    X = rng.integers(-3, 4, size=(n, d)).astype(np.float32)          # integers: plenty of equal values
    h = Harness(graph=(n, src, dst), X=X, model=tiny_model(kind, agg, dims, seed=d, hidden=16), dense_threshold=-1,
                precision="f32" if exact else "f64")
    ids = np.arange(2, n_src + 2, dtype=np.int32)
    h.feature_step(ids, rng.integers(-3, 4, size=(n_src, d)), exact=exact)
    # in one batch: removed, inserted and (from layer 2 on) changed edges of the hub
    k = n_src // 3
    new = rng.choice(np.arange(n_src + 2, n), size=k, replace=False)
    op = np.r_[np.full(k, DEL), np.full(2 * k, INS)].astype(np.uint8)
    bs = np.r_[ids[:k], new, np.full(k, n - 1)].astype(np.int32)
    bd = np.r_[np.zeros(2 * k), ids[k:2 * k]].astype(np.int32)
    h.step(op, bs, bd, exact=exact)
    h.check_state(exact=exact)
    h.ink.close()


def check_lengths(kind, agg, d, n_src, fan, n_dst):
    """Targets with 63 to 300 events, around every limit and chunk, among n_src * fan events on n_dst nodes."""
    n, lengths = n_src + n_dst, (63, 64, 65, 127, 128, 129, 192, 193, 255, 256, 257, 300)
    rng = np.random.default_rng(n_src + d)
    s = np.arange(n_src)
    src = [np.repeat(s, fan)] + [rng.choice(s, size=k, replace=False) for k in lengths]
    dst = [rng.integers(n_src + 20, n, size=n_src * fan)] + [np.full(k, n_src + i) for i, k in enumerate(lengths)]
    keys = np.unique(synth.edge_keys(np.concatenate(src).astype(np.int32), np.concatenate(dst).astype(np.int32)))
    src, dst = synth.keys_to_edges(keys)
    exact = agg in ("max", "min")
    X = rng.integers(-3, 4, size=(n, d)).astype(np.float32)
    h = Harness(graph=(n, src, dst), X=X, model=tiny_model(kind, agg, (d, 24, 6), seed=d, hidden=16), dense_threshold=-1,
                precision="f32" if exact else "f64")
    h.feature_step(s.astype(np.int32), rng.integers(-3, 4, size=(n_src, d)), exact=exact)
    assert h.ink.stats()["layers"][0]["n_events"] == len(src)
    h.check_state(exact=exact)
    h.ink.close()


SELECT_AND_SUM = [("sage", "max", 100), ("sage", "min", 20), ("gin", "sum", 40)]


@pytest.mark.parametrize("kind,agg,d", SELECT_AND_SUM)
@pytest.mark.parametrize("n_src,fan", [(1500, 190), (6000, 190)])     # 285 000 and 1 140 000 events in one layer
def test_limits_of_mid_size_launches(kind, agg, d, n_src, fan):
    """Many events a target: cut from 257 on."""
    check_lengths(kind, agg, d, n_src, fan, 12000)


@pytest.mark.parametrize("kind,agg,d", SELECT_AND_SUM)
@pytest.mark.parametrize("n_src,n_dst", [(1500, 60000), (1500, 30000), (6000, 120000)])
def test_low_limits_of_mid_size_launches(kind, agg, d, n_src, n_dst):
    """5 events a target, up to a million of them: cut from 65 on; 10: from 129 on."""
    check_lengths(kind, agg, d, n_src, 190, n_dst)
