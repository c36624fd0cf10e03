"""Sums of few rows: long rows are taken from 33 neighbours on, in chunks of 1024 that many waves share, and in slices of
32 columns.  Lengths around both limits and widths around whole slices, over all nodes of a graph that is small enough."""
import numpy as np
import pytest

import synth
from util import Harness
from test_gpu_edge_cases import tiny_model, INS, DEL

pytestmark = pytest.mark.gpu
LENGTHS = np.r_[np.arange(0, 300, 7), 31, 32, 33, 63, 64, 65, 127, 128, 129, 1023, 1024, 1025, 2047, 2048, 2049, 3073, 7700]


@pytest.mark.parametrize("kind,agg,d", [("sage", "sum", 3), ("sage", "mean", 32), ("gin", "sum", 33), ("sage", "mean", 48), ("gin", "sum", 52),
                                        ("sage", "mean", 64), ("gcn", "gcn_sym", 97), ("gin", "sum", 128), ("sage", "sum", 250), ("sage", "mean", 301)])
def test_long_rows_in_short_launches(kind, agg, d):
    n = 8192
    rng = np.random.default_rng(d)
    src = np.concatenate([rng.choice(n - 100, size=k, replace=False) + 100 for k in LENGTHS])
    dst = np.repeat(np.arange(LENGTHS.size), LENGTHS)
    src, dst = synth.keys_to_edges(np.unique(synth.edge_keys(src.astype(np.int32), dst.astype(np.int32))))
    X = rng.standard_normal((n, d)).astype(np.float32)
    dims = (9, d, 6) if kind == "gcn" else (d, 6)
    h = Harness(graph=(n, src, dst), X=X[:, :dims[0]].copy(), model=tiny_model(kind, agg, dims, seed=d, hidden=16), precision="f64",
                dense_threshold=1e-6)
    h.check_state(exact=False)
    gone = rng.choice(src.size, size=40, replace=False)               # and with every row summed again after a batch
    op = np.r_[np.full(40, DEL), np.full(2, INS)].astype(np.uint8)
    bs = np.r_[src[gone], [5, 6]].astype(np.int32)
    bd = np.r_[dst[gone], [n - 1, n - 2]].astype(np.int32)
    h.step(op, bs, bd, exact=False)
    h.check_state(exact=False)
    h.ink.close()


@pytest.mark.parametrize("kind,agg,d", [("sage", "sum", 129), ("gin", "sum", 200), ("sage", "mean", 256), ("gcn", "gcn_sym", 250)])
def test_events_of_wide_rows(kind, agg, d):
    """Every number of events a target that its last batches can leave over, around the window of 64, of changed, removed
    and inserted edges."""
    n, k = 3000, np.r_[np.arange(1, 27), 63, 64, 65, 66, 100, 127]
    rng = np.random.default_rng(d)
    src = np.concatenate([rng.choice(200, size=c, replace=False) for c in k])
    dst = np.repeat(1000 + np.arange(k.size), k)
    src, dst = synth.keys_to_edges(np.unique(synth.edge_keys(src.astype(np.int32), dst.astype(np.int32))))
    dims = (9, d, 6) if kind == "gcn" else (d, 12, 6)
    X = rng.standard_normal((n, dims[0])).astype(np.float32)
    h = Harness(graph=(n, src, dst), X=X, model=tiny_model(kind, agg, dims, seed=d, hidden=16), precision="f64", dense_threshold=-1)
    h.feature_step(np.arange(200, dtype=np.int32), rng.standard_normal((200, dims[0])).astype(np.float32), exact=False)
    h.check_state(exact=False)
    gone = np.unique(dst, return_index=True)[1]                        # one edge of every target goes and another comes
    op = np.r_[np.full(k.size, DEL), np.full(k.size, INS)].astype(np.uint8)
    bs = np.r_[src[gone], 300 + np.arange(k.size)].astype(np.int32)
    h.step(op, bs, np.r_[dst[gone], dst[gone]].astype(np.int32), exact=False)
    h.check_state(exact=False)
    h.ink.close()


@pytest.mark.parametrize("d,n", [(64, 2 ** 23 + 9), (128, 2 ** 22 + 9), (256, 2 ** 21 + 9)])
def test_long_rows_of_a_table_beyond_2_gib(d, n):
    """Whole rows instead of slices.  Terms are positive and no sum is more than 1024 additions deep in a lane group plus 3
    waves, 17 chunks and 2 groups: 1100 roundings of 2 ** -24 at most."""
    from paper_2309_11071_amd import Ink
    lengths = [1024, 1025, 2047, 2048, 2049, 4097, 33001]
    rng = np.random.default_rng(d)
    rowptr = np.zeros(n + 1, np.int64)
    rowptr[1:len(lengths) + 1] = np.cumsum(lengths)
    rowptr[len(lengths) + 1:] = rowptr[len(lengths)]
    col = np.concatenate([np.sort(rng.choice(n - 100, size=k, replace=False) + 100) for k in lengths]).astype(np.int32)
    base = rng.random((2 ** 14, d), dtype=np.float32)
    X = np.resize(base, (n, d))
    ink = Ink(rowptr, col, X, tiny_model("sage", "sum", (d, 3), seed=d))
    ink.full_infer()
    got = ink.get_layer(1, 1, 0, len(lengths) + 1)
    ink.close()
    for i, k in enumerate(lengths):
        want = X[col[rowptr[i]:rowptr[i + 1]]].astype(np.float64).sum(0)
        assert (np.abs(got[i] - want) <= 1100 * 2.0 ** -24 * want).all(), k
    assert (got[len(lengths)] == 0).all()


def chained_sum(x, groups):
    """fp32 sum of the rows of x as long rows are added: chunks of 1024, four parts of a chunk, `groups` chains in each part."""
    def chain(rows):
        return np.add.accumulate(rows, axis=0, dtype=np.float32)[-1] if len(rows) else np.zeros(x.shape[1], np.float32)
    chunks = []
    for c0 in range(0, len(x), 1024):
        c = x[c0:c0 + 1024]
        parts = [c[len(c) * w // 4:len(c) * (w + 1) // 4] for w in range(4)]
        chunks.append(chain(np.stack([chain(np.stack([chain(p[g::groups]) for g in range(groups)])) for p in parts])))
    return chain(np.stack([chain(np.stack(chunks[g::groups])) for g in range(min(groups, len(chunks)))]))


@pytest.mark.parametrize("d", [12, 41, 48])
def test_long_narrow_rows_are_as_exact_as_chains_of_51(d):
    """Errors against 64 bits, rms over 60 rows of 2000 to 6000 terms: those of the chains above.  An rms over 60 d values of which each
    is the end of a random walk has a spread of 1 / sqrt(120 d), 2.6 % for 12 columns; twice as long chains are a fifth worse."""
    from paper_2309_11071_amd import Ink
    n, rng = 9000, np.random.default_rng(d)
    lengths = np.zeros(n, np.int64)
    lengths[:60] = np.linspace(2000, 6000, 60)
    rowptr = np.r_[0, np.cumsum(lengths)]
    col = np.concatenate([np.sort(rng.choice(n - 60, size=k, replace=False) + 60) for k in lengths[:60]]).astype(np.int32)
    X = rng.standard_normal((n, d)).astype(np.float32)
    ink = Ink(rowptr, col, X, tiny_model("sage", "sum", (d, 3), seed=d))
    ink.full_infer()
    got = ink.get_layer(1, 1, 0, 60).astype(np.float64)
    ink.close()
    rows = [X[col[rowptr[i]:rowptr[i + 1]]] for i in range(60)]
    want = np.stack([r.astype(np.float64).sum(0) for r in rows])
    chains = np.stack([chained_sum(r, 5) for r in rows])
    rms = lambda e: float(np.sqrt((e ** 2).mean()))  # noqa: E731
    print("rms error %.3e, of the chains %.3e" % (rms(got - want), rms(chains - want)))
    assert rms(got - want) <= (1 + 3 / np.sqrt(120 * d)) * rms(chains - want)
