"""Small updates whose graph stage and layers run in one workgroup each: around the limit of 32 entries and events, widths at the edges of the lane
groups and of the transform's tiles, rows with many neighbours on both sides of what the workgroup recomputes itself,
updates whose later layers are too large for it, and batches without effect."""
import numpy as np
import pytest

import synth
from util import Harness
from test_gpu_edge_cases import tiny_model, INS, DEL

pytestmark = pytest.mark.gpu


def ring_with_hub(n, hub_deg, seed):
    """A ring with two chords per node, and node 0 with hub_deg in-neighbours."""
    v = np.arange(n)
    src = np.r_[v, v, v, np.arange(1, hub_deg + 1)]
    dst = np.r_[(v + 1) % n, (v + 17) % n, (v + n // 2) % n, np.zeros(hub_deg, np.int64)]
    keep = src != dst
    keys = np.unique(synth.edge_keys(src[keep].astype(np.int32), dst[keep].astype(np.int32)))
    return synth.keys_to_edges(keys)


@pytest.mark.parametrize("agg,dims", [("max", (20, 12, 6)), ("min", (64, 65, 32)), ("max", (100, 250, 7)), ("max", (256, 33, 129)),
                                      ("min", (128, 128, 128, 128)), ("max", (7, 256, 40))])
def test_small_updates(agg, dims):
    n = 6000
    src, dst = ring_with_hub(n, 300, dims[0])
    rng = np.random.default_rng(dims[1])
    X = rng.integers(-3, 4, size=(n, dims[0])).astype(np.float32)
    h = Harness(graph=(n, src, dst), X=X, model=tiny_model("sage", agg, dims, seed=dims[0]), precision="f32", slack=0.1)
    for size in (1, 2, 5, 15, 17, 31, 32, 33, 64, 1):
        s0, d0 = synth.keys_to_edges(h.keys)
        k = size // 2
        pick = rng.choice(s0.size, size=k, replace=False)
        op = np.r_[np.full(k, DEL), np.full(size - k, INS)].astype(np.uint8)
        s = np.r_[s0[pick], rng.integers(0, n, size=size - k)].astype(np.int32)
        d = np.r_[d0[pick], rng.integers(0, n, size=size - k)].astype(np.int32)
        h.step(op, s, d)
        h.step(op, s, d)                                          # again: no entry has an effect
        h.step((1 - op)[::-1].copy(), s[::-1].copy(), d[::-1].copy())
    h.check_state(); h.check_graph(); h.check_bound()
    h.ink.close()


@pytest.mark.parametrize("d,hub_deg", [(16, 900), (128, 4095), (128, 4500), (256, 2040), (256, 5000), (3, 20000)])
def test_exposed_hub(d, hub_deg):
    """The hub loses the neighbour that holds every dimension and has no recorded runner-up left."""
    n = hub_deg + 500
    src, dst = ring_with_hub(n, hub_deg, d)
    X = np.random.default_rng(hub_deg).uniform(0, 1, size=(n, d)).astype(np.float32)
    X[7] = 5.0; X[9] = 4.0; X[11] = 3.0
    h = Harness(graph=(n, src, dst), X=X, model=tiny_model("sage", "max", (d, 8, 5), seed=d), precision="f32")
    one = lambda op, u: h.step(np.array([op], np.uint8), np.array([u], np.int32), np.zeros(1, np.int32))
    for u in (7, 9, 11, 12):
        one(DEL, u)
    assert h.ink.stats()["layers"][0]["n_events"] == 1
    one(INS, 7)
    one(DEL, 7)
    h.check_state(); h.check_graph()
    h.ink.close()


def test_graph_store():
    """Blocks that move, with and without room in the pool, and all kinds of entries on few nodes."""
    n = 2000
    src, dst = ring_with_hub(n, 40, 1)
    X = np.random.default_rng(2).standard_normal((n, 12)).astype(np.float32)
    h = Harness(graph=(n, src, dst), X=X, model=tiny_model("sage", "max", (12, 9, 5), seed=4), precision="f32", slack=0.0, pool_reserve=300)
    rng = np.random.default_rng(3)
    for it in range(40):
        size = int(rng.integers(1, 33))
        s = rng.integers(0, 12, size=size).astype(np.int32)           # duplicates, self loops, no-ops
        d = rng.integers(0, 3 + it, size=size).astype(np.int32)
        h.step(rng.integers(0, 2, size=size).astype(np.uint8), s, d)
        s = rng.integers(0, n, size=30).astype(np.int32)
        h.step(np.full(30, INS, np.uint8), s, np.full(30, it, np.int32))
        h.step(np.full(30, DEL, np.uint8), np.full(30, it, np.int32), s)
    h.check_state(); h.check_graph()
    h.ink.close()


@pytest.mark.parametrize("hub_deg", [2 * 2048, 255 * 2048, 257 * 2048])
def test_long_block_to_walk(hub_deg):
    n = hub_deg + 50
    v = np.arange(1, hub_deg + 1)
    keys = np.unique(synth.edge_keys(v.astype(np.int32), np.zeros(hub_deg, np.int32)))
    src, dst = synth.keys_to_edges(keys)
    X = np.random.default_rng(1).uniform(0, 1, size=(n, 4)).astype(np.float32)
    h = Harness(graph=(n, src, dst), X=X, model=tiny_model("sage", "max", (4, 3, 2), seed=2), precision="f32")
    for op, u in ((DEL, hub_deg), (INS, hub_deg + 3), (DEL, 1), (INS, hub_deg), (INS, hub_deg)):
        h.step(np.array([op, INS], np.uint8), np.array([u, 3], np.int32), np.array([0, 5], np.int32))
    h.check_state(); h.check_graph()
    h.ink.close()


def test_bad_entries_leave_everything_untouched():
    from paper_2309_11071_amd.binding import InkError
    import torch
    n = 500
    src, dst = ring_with_hub(n, 20, 1)
    X = np.random.default_rng(2).standard_normal((n, 6)).astype(np.float32)
    h = Harness(graph=(n, src, dst), X=X, model=tiny_model("sage", "max", (6, 5, 4), seed=4), precision="f32")
    from paper_2309_11071_amd import Ink
    from paper_2309_11071_amd.binding import make_updates
    rp, col = h.ink.get_graph()
    dev = Ink(rp, col, X, h.model, batch_device=True)
    dev.full_infer()
    for op, s, d in (([0, 2], [1, 2], [3, 4]), ([0, 1], [1, n], [3, 4]), ([1, 0], [1, 2], [-1, 4])):
        t = torch.from_numpy(make_updates(np.array(op, np.uint8), np.array(s, np.int32), np.array(d, np.int32)).view(np.uint8).copy()).cuda()
        torch.cuda.synchronize()
        with pytest.raises(InkError):
            dev.apply_updates_device(t.data_ptr(), 2)
    assert np.array_equal(dev.get_graph()[1], col)
    t = torch.from_numpy(make_updates(np.array([0], np.uint8), np.array([3], np.int32), np.array([9], np.int32)).view(np.uint8).copy()).cuda()
    torch.cuda.synchronize()
    r = dev.apply_updates_device(t.data_ptr(), 1)
    h.step(np.array([0], np.uint8), np.array([3], np.int32), np.array([9], np.int32))
    assert r["n_applied_ins"] == 1
    for l in (1, 2):
        assert np.array_equal(dev.get_layer(l, 0).view(np.uint32), h.ink.get_layer(l, 0).view(np.uint32))
    dev.close(); h.ink.close()


@pytest.mark.parametrize("agg,dims", [("max", (256, 128, 90)), ("min", (250, 96, 256, 20)), ("max", (130, 20, 64, 64, 64, 64, 64, 33, 9))])
def test_products_handed_from_wave_to_wave(agg, dims):
    """Two to eight waves a tile, one to four blocks of k, waves that take a second block; the most layers there can be.
    One edge, the most rows of one tile (16 targets and sources) and one more."""
    n = 4000
    src, dst = ring_with_hub(n, 300, dims[1])
    rng = np.random.default_rng(dims[0])
    X = rng.integers(-3, 4, size=(n, dims[0])).astype(np.float32)
    h = Harness(graph=(n, src, dst), X=X, model=tiny_model("sage", agg, dims, seed=dims[1]), precision="f32")
    for size in (1, 3, 16, 17, 1):
        s, d = rng.integers(0, n, size=size).astype(np.int32), rng.choice(n, size=size, replace=False).astype(np.int32)
        h.step(np.full(size, INS, np.uint8), s, d)
        h.step(np.full(size, DEL, np.uint8), s[::-1].copy(), d[::-1].copy())
    h.check_state(); h.check_graph()
    h.ink.close()
