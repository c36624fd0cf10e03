"""Results copied to the host (ink_copy_result): by the gather itself and by a copy, widths with and without whole
16-byte groups, empty results, results too large for the pinned buffer, and what is refused."""
import numpy as np
import pytest

import synth
from paper_2309_11071_amd.binding import InkError, make_updates
from util import Harness
from test_gpu_edge_cases import tiny_model, INS, DEL

pytestmark = pytest.mark.gpu


def device_rows(r, d):
    import torch
    from paper_2309_11071_amd.binding import _dtoh
    ids, emb = np.empty(r["n_changed"], np.int32), np.empty((r["n_changed"], d), np.float32)
    _dtoh(ids, r["changed_ids_ptr"]); _dtoh(emb, r["embeddings_ptr"])
    return ids, emb


@pytest.mark.parametrize("agg,dout", [("max", 1), ("max", 7), ("min", 64), ("mean", 5), ("sum", 12), ("max", 256)])
def test_results_on_the_host(agg, dout):
    n, fan = 6000, 40
    rng = np.random.default_rng(dout)
    keys = np.unique(synth.edge_keys(rng.integers(0, n, n * fan).astype(np.int32), rng.integers(0, n, n * fan).astype(np.int32)))
    src, dst = synth.keys_to_edges(keys)
    src, dst = src[src != dst], dst[src != dst]
    X = rng.standard_normal((n, 12)).astype(np.float32)
    h = Harness(graph=(n, src, dst), X=X, model=tiny_model("sage", agg, (12, 9, dout), seed=dout),
                precision="f32" if agg in ("max", "min") else "f64")
    for size in (1, 1, 3, 40, 40, 2000, 2000, 1):            # one workgroup, short and long layers, beyond the pinned buffer at 256 columns
        pick = rng.choice(h.keys.size, size=size, replace=False)
        s, d = synth.keys_to_edges(h.keys[pick])
        for op in (DEL, INS):
            r = h.ink.apply_updates(make_updates(np.full(size, op, np.uint8), s.astype(np.int32), d.astype(np.int32)))
            ids, emb = device_rows(r, dout)
            assert np.array_equal(r["changed_ids"], ids) and np.array_equal(r["embeddings"].view(np.uint32), emb.view(np.uint32))
            if size == 40:                                   # a result that is not fetched, then one that is
                h.ink.apply_updates(make_updates(np.full(size, 1 - op, np.uint8), s.astype(np.int32), d.astype(np.int32)), fetch=False)
                h.ink.apply_updates(make_updates(np.full(size, op, np.uint8), s.astype(np.int32), d.astype(np.int32)), fetch=False)
    r = h.ink.update_features(np.arange(50, dtype=np.int32), rng.standard_normal((50, 12)).astype(np.float32))
    ids, emb = device_rows(r, dout)
    assert np.array_equal(r["changed_ids"], ids) and np.array_equal(r["embeddings"].view(np.uint32), emb.view(np.uint32))
    r = h.ink.apply_updates(make_updates([INS], [3], [3]))   # a self loop: nothing changes
    assert r["n_changed"] == 0 and r["changed_ids"].size == 0
    with pytest.raises(InkError):
        h.ink._fetch(1)
    h.ink.full_infer()
    with pytest.raises(InkError):
        h.ink._fetch(0)
    h.ink.close()


@pytest.mark.parametrize("refused", ["op", "id", "feature id", "infer"])
def test_nothing_is_left_behind_a_refused_call(refused):
    """A call that tried to change the context and was refused takes the last result with it, as the header says."""
    n = 300
    rng = np.random.default_rng(4)
    dst = np.arange(1, n, dtype=np.int32)
    h = Harness(graph=(n, dst - 1, dst), X=rng.standard_normal((n, 4)).astype(np.float32), model=tiny_model("sage", "max", (4, 3), seed=1))
    r = h.ink.apply_updates(make_updates([INS], [5], [3]))
    assert r["n_changed"] > 0
    h.ink._fetch(r["n_changed"])                             # as often as one likes
    if refused == "infer":
        h.ink.full_infer_noalloc()
    else:
        with pytest.raises(InkError):
            if refused == "feature id":
                h.ink.update_features(np.array([n], np.int32), np.ones((1, 4), np.float32))
            else:
                h.ink.apply_updates(make_updates([2 if refused == "op" else INS], [5], [n if refused == "id" else 4]))
    with pytest.raises(InkError) as e:
        h.ink._fetch(r["n_changed"])
    assert e.value.status == 2
    h.ink.close()


def test_nothing_is_left_behind_a_refused_inference():
    from paper_2309_11071_amd import Ink
    n, rng = 200_000, np.random.default_rng(5)               # staging rows of 128 floats for every node: more than the static array holds
    dst = np.arange(1, n, dtype=np.int32)
    ink = Ink(*synth.in_csr_from_edges(n, dst - 1, dst), rng.standard_normal((n, 4)).astype(np.float32), tiny_model("gin", "sum", (4, 3), seed=1, hidden=128))
    ink.full_infer()
    r = ink.update_features(np.arange(4, dtype=np.int32), np.ones((4, 4), np.float32))
    assert r["n_changed"] > 0
    with pytest.raises(InkError) as e:
        ink.full_infer_noalloc()
    assert e.value.status == 5
    with pytest.raises(InkError) as e:
        ink._fetch(r["n_changed"])
    assert e.value.status == 2
    ink.close()
