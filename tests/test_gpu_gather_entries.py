"""The gather of max / min recomputes orders entries (value, id) as doubles: values whose bits are not ordered as the
values are (zeros of both signs, the smallest subnormal numbers, both infinities) in rows of every kind of length."""
import numpy as np
import pytest

import oracle
import synth
from test_gpu_edge_cases import tiny_model

pytestmark = pytest.mark.gpu
F = np.float32
TINY = np.array([1], np.uint32).view(F)[0]
VALUES = np.array([0.0, -0.0, TINY, -TINY, 1.0, -1.0, np.finfo(F).tiny, -np.finfo(F).tiny], F)


def reference(rp, col, X, is_min):
    """value, holder, runner-up value, runner-up id per node and column: equal values (zeros of either sign) go by the id"""
    n, d = rp.size - 1, X.shape[1]
    worst = F(np.inf if is_min else -np.inf)
    out = [np.zeros((n, d), F), np.full((n, d), -1, np.int32), np.full((n, d), worst, F), np.full((n, d), -1, np.int32)]
    for v in range(n):
        nb = col[rp[v]:rp[v + 1]]              # ascending
        rows = X[nb]
        order = np.argsort(rows if is_min else -rows, axis=0, kind="stable")     # -0 == 0 here, too
        for k in range(min(2, nb.size)):
            pick = order[k]
            val, ids = np.take_along_axis(rows, pick[None], 0)[0], nb[pick]
            taken = val != worst               # the worst infinity takes no place in a list that is ascending
            out[2 * k][v] = np.where(taken, val, out[2 * k][v])
            out[2 * k + 1][v] = np.where(taken, ids, -1)
    return out


@pytest.mark.parametrize("agg,d", [("max", 12), ("min", 64), ("max", 128), ("min", 100), ("max", 250), ("min", 300)])
@pytest.mark.parametrize("inf", [False, True])
def test_special_values(agg, d, inf):
    from paper_2309_11071_amd import Ink
    rng = np.random.default_rng(d)
    lengths = np.r_[np.arange(140), 255, 256, 257, 300, 1023, 1030, 3000]
    for n in (9000, 5000):                     # more and fewer targets than a short launch has
        dst = np.repeat(np.arange(lengths.size), lengths)
        src = np.concatenate([rng.choice(n - 200, size=k, replace=False) + 200 for k in lengths])
        keys = np.unique(synth.edge_keys(src.astype(np.int32), dst.astype(np.int32)))
        rp, col = oracle.csr_from_keys(n, keys)
        X = rng.choice(VALUES, size=(n, d))
        if inf:                                # rows with no, some and only infinite entries
            X[rng.random((n, d)) < 0.5] = np.inf
            X[rng.random((n, d)) < 0.5] = -np.inf
        ink = Ink(rp, col, X, tiny_model("sage", agg, (d, 4), seed=3))
        ink.full_infer()
        want = reference(rp, col, X, agg == "min")
        for which in (1, 2, 3, 4):
            got = ink.get_layer(1, which)
            assert np.array_equal(got.view(np.uint32), want[which - 1].view(np.uint32)), (n, which)
        ink.close()


NANS = np.array([0x7f800001, 0x7fc00000, 0x7fe00000, 0x7fefffff, 0x7ff00000, 0x7ff00001, 0x7ff7ffff, 0x7ff80000, 0x7fffffff,
                 0xff800001, 0xffc00000, 0xffe00000, 0xffefffff, 0xfff00000, 0xfff00001, 0xfff7ffff, 0xfff80000, 0xffffffff], np.uint32).view(F)


@pytest.mark.parametrize("agg,d", [("max", 12), ("min", 64), ("max", 128), ("min", 100), ("max", 250), ("min", 300)])
def test_a_nan_takes_no_place(agg, d):
    """NaNs of every kind that the bits of a double can be made of (none, quiet, signalling), few, many, and nothing else"""
    from paper_2309_11071_amd import Ink
    from paper_2309_11071_amd.binding import make_updates
    rng = np.random.default_rng(d)
    lengths = np.r_[np.arange(70), 127, 128, 129, 300, 1030, 3000]
    for n in (9000, 5000):
        dst = np.repeat(np.arange(lengths.size), lengths)
        src = np.concatenate([rng.choice(n - 200, size=k, replace=False) + 200 for k in lengths])
        rp, col = oracle.csr_from_keys(n, np.unique(synth.edge_keys(src.astype(np.int32), dst.astype(np.int32))))
        for share in (0.02, 0.5, 1.0):
            X = rng.standard_normal((n, d)).astype(F)
            nan = rng.random((n, d)) < share
            X[nan] = rng.choice(NANS, size=int(nan.sum()))
            ink = Ink(rp, col, X, tiny_model("sage", agg, (d, 4), seed=3))
            ink.full_infer()
            want = reference(rp, col, np.where(np.isnan(X), F(np.inf if agg == "min" else -np.inf), X), agg == "min")
            for which in (1, 2, 3, 4):
                got = ink.get_layer(1, which)
                assert np.array_equal(got.view(np.uint32), want[which - 1].view(np.uint32)), (n, share, which)
            keys = synth.edge_keys(col, np.repeat(np.arange(n, dtype=np.int32), np.diff(rp)))
            for size in (20, 400):             # edges that go: rows gathered by the kernels that reduce a target's events
                gone = rng.choice(keys.size, size=size, replace=False)
                s, t = synth.keys_to_edges(keys[gone])
                ink.apply_updates(make_updates(np.full(size, 1, np.uint8), s.astype(np.int32), t.astype(np.int32)))
                keys = np.delete(keys, gone)
                want = reference(*oracle.csr_from_keys(n, keys), np.where(np.isnan(X), F(np.inf if agg == "min" else -np.inf), X), agg == "min")
                for which in (1, 2):
                    got = ink.get_layer(1, which)
                    assert np.array_equal(got.view(np.uint32), want[which - 1].view(np.uint32)), (n, share, size, which)
            ink.close()


def test_no_nan_behind_a_relu():
    """What lets the gathers of later layers look for none: rows of a layer that ends in ReLU have no NaN and no sign bit, in an inference
    and in updates of few and of many rows."""
    from paper_2309_11071_amd import Ink
    n, d, rng = 5000, 12, np.random.default_rng(2)
    dst = rng.integers(0, n, 4 * n).astype(np.int32)
    src = ((dst + 1 + rng.integers(0, n - 1, dst.size)) % n).astype(np.int32)
    X = rng.standard_normal((n, d)).astype(F)
    X[rng.random((n, d)) < 0.05] = NANS[0]
    ink = Ink(*oracle.csr_from_keys(n, np.unique(synth.edge_keys(src, dst))), X, tiny_model("sage", "max", (d, 8, 4), seed=3))
    ink.full_infer()
    for rows in (0, 3, 2000):
        if rows:
            Y = rng.standard_normal((rows, d)).astype(F)
            Y[rng.random((rows, d)) < 0.2] = rng.choice(NANS)
            ink.update_features(rng.choice(n, size=rows, replace=False).astype(np.int32), Y)
        got = ink.get_layer(1, 0)
        assert not np.isnan(got).any() and not np.signbit(got).any() and (got > 0).any()
    ink.close()
