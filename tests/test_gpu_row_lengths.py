"""Rows of every length that matters to the gathers: all of 0 .. 330 in-neighbours (batches, windows of 60 and 64 ids, the
limits of the long-row path), lengths around its chunks of 1024, and rows of up to 70 chunks, at every lane width; and
the copy of a table's rows to the caller at widths and addresses with and without whole 16-byte groups."""
import numpy as np
import pytest

import synth
from util import Harness
from test_gpu_edge_cases import tiny_model, INS

pytestmark = pytest.mark.gpu
LONG = [511, 512, 1023, 1024, 1025, 2047, 2049, 4096, 4097, 8193, 33000, 71000]


@pytest.mark.parametrize("agg,d", [("max", 12), ("min", 64), ("max", 100), ("min", 128), ("max", 250), ("max", 300), ("sum", 7), ("sum", 44),
                                   ("mean", 64), ("sum", 128), ("mean", 121), ("sum", 256), ("sum", 300)])
def test_row_lengths(agg, d):
    n = 72000
    rng = np.random.default_rng(d)
    lengths = np.r_[np.arange(331), LONG]
    src = np.concatenate([rng.choice(n - 1000, size=k, replace=False) + 1000 for k in lengths])
    dst = np.repeat(np.arange(lengths.size), lengths)
    src, dst = synth.keys_to_edges(np.unique(synth.edge_keys(src.astype(np.int32), dst.astype(np.int32))))
    exact = agg in ("max", "min")
    X = rng.integers(-3, 4, size=(n, d)).astype(np.float32) if exact else rng.standard_normal((n, d)).astype(np.float32)
    h = Harness(graph=(n, src, dst), X=X, model=tiny_model("sage", agg, (d, 6), seed=d), precision="f32" if exact else "f64")
    h.check_state(exact=exact)
    if exact:                                 # lists that are no longer ascending, all rows again
        v = np.arange(lengths.size, dtype=np.int32)
        h.step(np.full(v.size, INS, np.uint8), (v % 600 + 343).astype(np.int32), v)
        h.ink.full_infer()
        h.check_state(); h.check_bound(exact=True, max_nodes=n)
    h.ink.close()


@pytest.mark.parametrize("d", [3, 4, 44, 128, 301])
def test_rows_to_the_caller(d):
    import torch
    from paper_2309_11071_amd.binding import load_library
    n = 5000
    X = np.random.default_rng(d).standard_normal((n, d)).astype(np.float32)
    h = Harness(graph=(n, np.array([1], np.int32), np.array([0], np.int32)), X=X, model=tiny_model("sage", "max", (d, 3), seed=1), precision="f32")
    for row0, rows, shift in ((0, n, 0), (17, 2049, 0), (4999, 1, 0), (3, 1000, 1)):
        out = torch.full((rows * d + 8,), 7.0, device="cuda")
        torch.cuda.synchronize()
        assert load_library().ink_get_layer(h.ink._h, 0, 0, row0, rows, out.data_ptr() + 4 * shift, 1, None) == 0
        got = out.cpu().numpy()
        assert np.array_equal(got[shift:shift + rows * d].reshape(rows, d), X[row0:row0 + rows])
        assert (got[:shift] == 7).all() and (got[shift + rows * d:] == 7).all()
    h.ink.close()
