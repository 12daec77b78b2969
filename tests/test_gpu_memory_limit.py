"""Rows and grouped incidences that indexes keep give way when memory runs out: under a limit on a context's
buffers, as many indexes are built and answered as when every call compares slots."""
import numpy as np
import pytest

import datagen
import oracle

torch = pytest.importorskip("torch")
bm = pytest.importorskip("paper_1102_1003_amd")

pytestmark = pytest.mark.gpu

M, N, P, LIMIT_MB = 200_000, 300, 0.02, 96


@pytest.fixture(scope="module")
def data():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    off, tids = datagen.bernoulli_sets(M, N, P, seed=1)
    rows, items = datagen.sets_to_transactions(M, off, tids)
    return off, tids, rows, items, oracle.all_pairs(off, tids)


def fill(data):
    """Builds indexes until one is refused, all pairs counted after each; the indexes and their context."""
    off, tids, rows, items, want = data
    ctx = bm.Context(0)
    held = []
    while len(held) < 64:
        try:
            ix = bm.Index.from_transactions(ctx, N, rows, items)
            assert np.array_equal(ix.all_pair_supports(), want)
        except bm.BatmapError as e:
            assert e.status == bm.BM_ENOMEM
            break
        held.append(ix)
    return ctx, held


@pytest.mark.parametrize("sparse", [False, True])
def test_as_many_indexes_as_by_slots(monkeypatch, data, sparse):
    off, tids, rows, items, want = data
    monkeypatch.setenv("BM_MEM_LIMIT_MB", str(LIMIT_MB))
    monkeypatch.setenv("BM_BIT_INGEST", "0")
    monkeypatch.setenv("BM_BITMAP_ROUTE", "0")
    ctx, held = fill(data)
    most = len(held)
    assert 1 < most < 64
    ctx.close()
    monkeypatch.setenv("BM_BIT_INGEST", "0" if sparse else "1")
    monkeypatch.setenv("BM_BITMAP_ROUTE", "2" if sparse else "1")
    ctx, held = fill(data)
    assert len(held) >= most
    for ix in held:                                          # rows gone or kept: the same counts
        assert np.array_equal(ix.all_pair_supports(), want)
        assert np.array_equal(ix.subset_pair_supports(np.arange(20)), oracle.subset_pairs(off, tids, np.arange(20)))
    ctx.close()


def test_rows_in_use_stay(monkeypatch, data):
    """A batch's, a server's and a graph's rows are not given back."""
    off, tids, rows, items, want = data
    monkeypatch.setenv("BM_MEM_LIMIT_MB", str(LIMIT_MB))
    monkeypatch.setenv("BM_BIT_INGEST", "1")
    monkeypatch.setenv("BM_BITMAP_ROUTE", "1")
    stream = torch.cuda.Stream()
    ctx = bm.Context(0, stream)
    a, b, c = (bm.Index.from_transactions(ctx, N, rows, items) for _ in range(3))
    outs = [torch.zeros(want.size, dtype=torch.int32, device="cuda:0") for _ in range(2)]
    torch.cuda.synchronize()
    batch = bm.Batch(ctx, [a], outs[:1])
    srv = bm.Server(b, streams=1, memory_budget=1 << 20)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream, capture_error_mode="thread_local"):
        c.all_pair_supports(outs[1])
    more = []
    with pytest.raises(bm.BatmapError) as e:
        while len(more) < 64:
            more.append(bm.Index.from_transactions(ctx, N, rows, items))
    assert e.value.status == bm.BM_ENOMEM
    for rep in range(2):
        for o in outs:
            o.fill_(-1)
        torch.cuda.synchronize()
        batch.run()
        g.replay()
        q = np.arange(10, 40, dtype=np.uint32)
        got, _ = srv.wait(srv.submit(q), timeout_s=60.0)
        assert np.array_equal(got, oracle.subset_pairs(off, tids, q))
        torch.cuda.synchronize()
        for o in outs:
            assert np.array_equal(o.cpu().numpy().view(np.uint32), want)
    del g
    batch.close()
    srv.close()
    ctx.close()
