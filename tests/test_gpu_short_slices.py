"""Long rows of launches over few nodes: in slices up to a number of chunks, whole rows beyond.  Numbers of rows around that line, for
widths of one to eight slices, rows of one chunk and of two."""
import numpy as np
import pytest

from test_gpu_edge_cases import tiny_model
from test_gpu_gather_entries import reference

pytestmark = pytest.mark.gpu
ITEMS = 512                        # chunks times slices of 32 columns
F = np.float32


def graph(rng, n, lengths):
    deg = np.zeros(n, np.int64)
    deg[rng.permutation(n)[:lengths.size]] = lengths
    dst = np.repeat(np.arange(n), deg)
    src = np.concatenate([np.sort(rng.choice(n - 1, size=k, replace=False)) for k in deg])
    return np.r_[0, np.cumsum(deg)], (src + (src >= dst)).astype(np.int32)


@pytest.mark.parametrize("agg,d", [(a, d) for a in ("max", "sum") for d in (30, 41, 64, 100, 128, 250)] + [("min", 129), ("mean", 256)])
def test_rows_around_the_line(agg, d):
    from paper_2309_11071_amd import Ink
    n, rng = 4000, np.random.default_rng(d)
    X = rng.standard_normal((n, d)).astype(F)
    chunks = ITEMS // ((d + 31) // 32)
    for rows in (1, chunks - 1, chunks, chunks + 1, 1200):
        lengths = rng.integers(130, 160, rows)
        lengths[0] = 1030                                      # two chunks: the line is crossed one row earlier
        rp, col = graph(rng, n, lengths)
        ink = Ink(rp, col, X, tiny_model("sage", agg, (d, 3), seed=1))
        ink.full_infer()
        if agg in ("max", "min"):
            want = reference(rp, col, X, agg == "min")
            for which in (1, 2, 3, 4):
                assert np.array_equal(ink.get_layer(1, which).view(np.uint32), want[which - 1].view(np.uint32)), (rows, which)
        else:
            got = ink.get_layer(1, 1).astype(np.float64)
            v = np.flatnonzero(np.diff(rp))
            want = np.add.reduceat(X[col].astype(np.float64), rp[v], axis=0)
            size = np.add.reduceat(np.abs(X[col]).astype(np.float64), rp[v], axis=0)
            # a chain of k fp32 additions errs by at most k 2^-24 of the sum of magnitudes; no chain of these rows has more than 80
            assert (np.abs(got[v] - want) <= 80 * 2.0 ** -24 * size).all(), rows
            assert not got[np.diff(rp) == 0].any()
        ink.close()


@pytest.mark.parametrize("agg,d", [("max", 41), ("max", 64), ("min", 128), ("max", 250), ("sum", 41), ("sum", 64), ("mean", 128), ("sum", 250)])
def test_parts_combined_by_the_last_or_by_a_kernel(agg, d):
    """Rows of one to four chunks, so many edges that the parts are expected to be the most that the last one combines, one more, which a kernel of
    its own combines, and many."""
    from paper_2309_11071_amd import Ink
    n, rng = 4200, np.random.default_rng(d)
    X = rng.standard_normal((n, d)).astype(F)
    line = 2048 if agg in ("sum", "mean") and d <= 128 else 256
    for expected in (line, line + 1, 2501):
        edges = next(e for e in range(0, 1 << 20, 128) if e // 1024 + min(n, e // 256) + 1 >= expected)
        assert edges // 1024 + min(n, edges // 256) + 1 == expected
        lengths = np.r_[1023, 1024, 1025, 2049, 4100, rng.integers(130, 160, n)]
        lengths = lengths[:np.searchsorted(np.cumsum(lengths), edges)]
        lengths = np.r_[lengths, edges - lengths.sum()]
        rp, col = graph(rng, n, lengths)
        ink = Ink(rp, col, X, tiny_model("sage", agg, (d, 3), seed=1))
        ink.full_infer()
        if agg in ("max", "min"):
            want = reference(rp, col, X, agg == "min")
            for which in (1, 2, 3, 4):
                assert np.array_equal(ink.get_layer(1, which).view(np.uint32), want[which - 1].view(np.uint32)), (expected, which)
        else:
            got = ink.get_layer(1, 1).astype(np.float64)
            v = np.flatnonzero(np.diff(rp))
            want = np.add.reduceat(X[col].astype(np.float64), rp[v], axis=0)
            size = np.add.reduceat(np.abs(X[col]).astype(np.float64), rp[v], axis=0)
            assert (np.abs(got[v] - want) <= 80 * 2.0 ** -24 * size).all(), expected       # as above: parts and their combination are short chains
            assert not got[np.diff(rp) == 0].any()
        ink.close()
