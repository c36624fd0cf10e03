"""What a caller may rely on when a call returns: the result is there for every stream, and after a rejected batch
nothing is left running on the context's own."""
import numpy as np
import pytest

from test_gpu_edge_cases import tiny_model
from test_gpu_layer_one import ring_with_hub

pytestmark = pytest.mark.gpu


def device_context(n, dims, **kw):
    import torch
    from paper_2309_11071_amd import Ink
    import synth
    src, dst = ring_with_hub(n, 200, 1)
    rp, col = synth.in_csr_from_edges(n, src, dst)
    X = np.random.default_rng(n).standard_normal((n, dims[0])).astype(np.float32)
    stream = torch.cuda.Stream()
    ink = Ink(rp, col, X, tiny_model("sage", "max", dims, seed=3), batch_device=True, stream=stream.cuda_stream, **kw)
    ink.full_infer()
    return ink, stream


def device_batch(op, s, d):
    import torch
    from paper_2309_11071_amd.binding import make_updates
    u = make_updates(np.asarray(op, np.uint8), np.asarray(s, np.int32), np.asarray(d, np.int32))
    t = torch.from_numpy(u.view(np.uint8).copy()).cuda()
    torch.cuda.synchronize()
    return t, u.size


@pytest.mark.parametrize("size", [1, 32, 33, 1024, 16384, 16385])        # both ends of each form of the graph stage
def test_rejected_batch_leaves_nothing_running(size):
    from paper_2309_11071_amd.binding import InkError
    n = 3000
    ink, stream = device_context(n, (16,) * 9)                           # 8 layers: the most that is enqueued ahead
    rng = np.random.default_rng(size)
    op, s, d = rng.integers(0, 2, size), rng.integers(0, n, size), rng.integers(0, n, size)
    s[size // 2] = n
    t, m = device_batch(op, s, d)
    running = 0
    for _ in range(50):
        with pytest.raises(InkError):
            ink.apply_updates_device(t.data_ptr(), m)
        running += not stream.query()
    assert running == 0
    ink.close()


@pytest.mark.parametrize("ids", [(5, 5), (5, 3000), (-1, 5)])
def test_rejected_features_leave_nothing_running(ids):
    import torch
    from paper_2309_11071_amd.binding import InkError
    ink, stream = device_context(3000, (16, 8))
    rows = torch.zeros(2, 16, device="cuda")
    t = torch.tensor(ids, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    running = 0
    for _ in range(50):
        with pytest.raises(InkError):
            ink.update_features_device(t.data_ptr(), rows.data_ptr(), 2)
        running += not stream.query()
    assert running == 0
    ink.close()


class Rows:
    def __init__(self, ptr, shape, typestr):
        self.__cuda_array_interface__ = dict(data=(ptr, False), shape=shape, typestr=typestr, version=3)


@pytest.mark.parametrize("size", [1, 200])       # layers of one workgroup, whose last writes the record itself; separate stages
@pytest.mark.parametrize("width", [8, 256])
def test_result_is_there_for_another_stream(size, width):
    import torch
    n = 3000
    ink, _ = device_context(n, (16, 16, width))
    other = torch.cuda.Stream()
    rng = np.random.default_rng(width)
    s, d = rng.integers(0, n, size), rng.integers(0, n, size)
    s[0], d[0] = 3, 9                             # not an edge of the graph
    batches = [device_batch(np.full(size, op), s, d) for op in (0, 1)]
    for i in range(100):
        t, m = batches[i % 2]
        r = ink.apply_updates_device(t.data_ptr(), m)
        k = r["n_changed"]
        assert k > 0
        with torch.cuda.stream(other):
            ids = torch.as_tensor(Rows(r["changed_ids_ptr"], (k,), "<i4"), device="cuda").clone()
            rows = torch.as_tensor(Rows(r["embeddings_ptr"], (k, width), "<f4"), device="cuda").clone()
        other.synchronize()
        assert np.array_equal(rows.cpu().numpy().view(np.uint32), ink.get_layer(2, 0)[ids.cpu().numpy()].view(np.uint32))
    ink.close()
