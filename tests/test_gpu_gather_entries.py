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
