"""The bitmap route on the GPU: bit rows and the Gram kernel at the edges of tiles, stages and
row segments, against the oracle's merge.  Counts are integers, so every comparison is exact."""
import numpy as np
import pytest

import datagen
import oracle

torch = pytest.importorskip("torch")
bm = pytest.importorskip("paper_1102_1003_amd")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = bm.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("tile", [0, 64, 128, 256])
@pytest.mark.parametrize("m,n,p", [
    (1, 2, 1.0), (31, 3, 0.5), (511, 63, 0.3), (512, 64, 0.3), (513, 65, 0.3),   # stage and tile edges
    (1024, 128, 0.1), (2000, 129, 0.1), (3000, 257, 0.1),
    (131_071, 40, 0.02), (131_072, 40, 0.9), (131_073, 40, 0.5),                 # row segment edges, dense rows
    (30_011, 613, 0.03), (400_000, 70, 0.01),
])
def test_dense_route(ctx, monkeypatch, tile, m, n, p):
    if tile:
        monkeypatch.setenv("BM_GRAM_TILE", str(tile))
    off, tids = datagen.bernoulli_sets(m, n, p, seed=m + n)
    idx = bm.Index.from_sets(ctx, m, off, tids)
    got = idx.all_pair_supports_dense(np.full(bm.n_pairs(n), 7, np.uint32))
    assert np.array_equal(got, oracle.all_pairs(off, tids))


def test_counts_past_fp32(ctx):
    """Full sets over more than 2^24 transactions: every count is m, which fp32 cannot hold."""
    m, n = 2**24 + 3, 3
    off = np.arange(n + 1, dtype=np.uint64) * m
    tids = np.tile(np.arange(m, dtype=np.uint32), n)
    idx = bm.Index.from_sets(ctx, m, off, tids)
    assert np.array_equal(idx.all_pair_supports_dense(), np.full(3, m, np.uint32))


@pytest.mark.parametrize("route", ["0", "1", "2", None])       # slots, bits, transactions, by time
@pytest.mark.parametrize("m,n,p,opts", [
    (10_000, 200, 0.02, {}),
    (20_000, 90, 0.3, dict(max_loop=0)),             # every insertion fails: slot counts are all corrections
    (60_000, 150, 0.002, dict(slot_bits=16)),
    (5_000, 2, 0.5, {}),
    (300_000, 1500, 0.0005, dict(slot_bits=0)),
    (1_000, 9000, 0.001, dict(slot_bits=0)),         # rows past 32 KB of counters
])
def test_pairs_either_route(ctx, monkeypatch, route, m, n, p, opts):
    """All pairs and frequent pairs give the same counts by slots, bits and transactions."""
    if route is not None:
        monkeypatch.setenv("BM_BITMAP_ROUTE", route)
    rng = np.random.default_rng(m)
    off, tids = datagen.sets_from_probs(m, p * rng.uniform(0, 2, n), seed=m + n)
    want = oracle.all_pairs(off, tids)
    sizes = np.sort(np.diff(off))
    idx = bm.Index.from_sets(ctx, m, off, tids, **opts)
    for rep in range(2):                               # rows made, rows kept
        assert np.array_equal(idx.all_pair_supports(np.full(want.size, 9, np.uint32)), want)
        ctx.set_profiling(True)
        idx.all_pair_supports()
        assert (ctx.timings()["compare_slot_pairs"] == 0) == (route in ("1", "2")) or route is None
        ctx.set_profiling(False)
    for sigma in (0, 1, int(np.median(want)) + 1, int(sizes[n // 2]), int(sizes[-1]), int(sizes[-1]) + 1):
        fresh = bm.Index.from_sets(ctx, m, off, tids, **opts)          # rows of the live items alone
        pruned = bm.Index.from_sets(ctx, m, off, tids, min_support=sigma, **opts)
        ref = oracle.frequent_pairs(off, tids, sigma)
        for ix in (idx, fresh, pruned):
            assert np.array_equal(ix.frequent_pairs(sigma), ref), sigma


def test_capture_takes_the_slot_compare(monkeypatch):
    """A captured call replays right after eager calls have made (and used) the bit rows."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    stream = torch.cuda.Stream()
    c = bm.Context(0, stream)
    m, n = 40_000, 300
    off, tids = datagen.bernoulli_sets(m, n, 0.05, seed=3)
    want = oracle.all_pairs(off, tids)
    idx = bm.Index.from_sets(c, m, off, tids)
    out = torch.zeros(want.size, dtype=torch.int32, device="cuda:0")
    monkeypatch.setenv("BM_BITMAP_ROUTE", "0")
    torch.cuda.synchronize()
    idx.all_pair_supports(out)                         # the slot compare's streams and events exist
    monkeypatch.setenv("BM_BITMAP_ROUTE", "1")
    idx.all_pair_supports(out)
    c.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream, capture_error_mode="thread_local"):
        idx.all_pair_supports(out)
    for rep in range(3):
        out.fill_(-1)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy().view(np.uint32), want)
        assert np.array_equal(idx.all_pair_supports(), want)
    del g
    c.close()


@pytest.mark.parametrize("route", ["0", "1", None])
def test_subsets_either_route(ctx, monkeypatch, route):
    """Subset queries in any order, on host and device buffers, while the index makes rows per query and
    then keeps them all; refused queries stay refused."""
    if route is not None:
        monkeypatch.setenv("BM_BITMAP_ROUTE", route)
    m, n = 20_000, 150
    rng = np.random.default_rng(7)
    off, tids = datagen.sets_from_probs(m, 0.1 * rng.uniform(0, 2, n), seed=8)
    idx = bm.Index.from_sets(ctx, m, off, tids)
    for k in (2, 3, 64, 65, 33, 100, 150, 40, 1):
        q = rng.choice(n, size=k, replace=False).astype(np.uint32)
        want = oracle.subset_pairs(off, tids, q)
        assert np.array_equal(idx.subset_pair_supports(q)[:want.size], want), k
        out = torch.full((max(want.size, 1),), -1, dtype=torch.int32, device="cuda:0")
        torch.cuda.synchronize()
        idx.subset_pair_supports(torch.from_numpy(q.view(np.int32)).to("cuda:0"), out)
        assert np.array_equal(out.cpu().numpy().view(np.uint32)[:want.size], want), k
    pruned = bm.Index.from_sets(ctx, m, off, tids, min_support=int(np.diff(off)[5]) + 1)
    for ix, q, code in ((idx, [1, 2, 1], bm.BM_EINVAL), (idx, [1, n], bm.BM_ERANGE), (pruned, [5, 6], bm.BM_EINVAL)):
        with pytest.raises(bm.BatmapError) as e:
            ix.subset_pair_supports(q)
        assert e.value.status == code


@pytest.mark.parametrize("route", ["0", "1", None])
@pytest.mark.parametrize("m,na,nb", [(5_000, 1, 1), (20_000, 65, 130), (3_000, 300, 3), (40_000, 64, 128)])
def test_cross_either_route(ctx, monkeypatch, route, m, na, nb):
    if route is not None:
        monkeypatch.setenv("BM_BITMAP_ROUTE", route)
    oa, ta = datagen.bernoulli_sets(m, na, 0.1, seed=m)
    ob, tb = datagen.bernoulli_sets(m, nb, 0.03, seed=m + 1)
    A, B = (bm.Index.from_sets(ctx, m, o, t, max_loop=2) for o, t in ((oa, ta), (ob, tb)))
    want = oracle.cross(oa, ta, ob, tb).reshape(na, nb)
    assert np.array_equal(bm.cross_pair_supports(A, B, np.full((na, nb), 5, np.uint32)), want)
    assert np.array_equal(bm.cross_pair_supports(B, A), want.T)
    sigma = max(1, int(np.median(want)))
    i, j = np.nonzero(want >= sigma)
    assert np.array_equal(bm.cross_pairs(A, B, sigma), np.stack([i, j, want[i, j]], 1))


@pytest.mark.parametrize("route", ["0", "1", None])
def test_batch_either_route(ctx, monkeypatch, route):
    """A batch of instances on both routes (None: the sparse one stays with slots), replayed between eager calls."""
    if route is not None:
        monkeypatch.setenv("BM_BITMAP_ROUTE", route)
    shapes = [(30_000, 400, 0.05), (200_000, 900, 0.0002), (500, 1, 0.5), (9_000, 65, 0.2), (12_000, 700, 0.03),
              (20_000, 130, 0.1), (50_000, 260, 0.02)]
    sets = [datagen.bernoulli_sets(m, n, p, seed=q) for q, (m, n, p) in enumerate(shapes)]
    idx = [bm.Index.from_sets(ctx, m, *s, max_loop=3) for (m, n, p), s in zip(shapes, sets)]
    want = [oracle.all_pairs(*s) for s in sets]
    outs = [torch.zeros(max(w.size, 1), dtype=torch.int32, device="cuda:0") for w in want]
    torch.cuda.synchronize()
    batch = bm.Batch(ctx, idx, outs)
    for rep in range(4):
        for o in outs:
            o.fill_(-1)
        torch.cuda.synchronize()
        batch.run()
        ctx.synchronize()
        for (m, n, p), o, w, ix in zip(shapes, outs, want, idx):
            assert np.array_equal(o.cpu().numpy().view(np.uint32)[:bm.n_pairs(n)], w[:bm.n_pairs(n)]), (m, n)
            assert np.array_equal(ix.all_pair_supports()[:bm.n_pairs(n)], w[:bm.n_pairs(n)])
    batch.close()


@pytest.mark.parametrize("tile", ["64", "128", "256"])
def test_joint_launch_tiles(ctx, monkeypatch, tile):
    """Families around tile edges in one launch (256: one launch each)."""
    monkeypatch.setenv("BM_BITMAP_ROUTE", "1")
    monkeypatch.setenv("BM_GRAM_TILE", tile)
    shapes = [(511, 2), (70_000, 64), (513, 65), (30_000, 128), (10_000, 257), (1, 3), (40_000, 129)]
    sets = [datagen.bernoulli_sets(m, n, 0.3, seed=50 + q) for q, (m, n) in enumerate(shapes)]
    idx = [bm.Index.from_sets(ctx, m, *s) for (m, n), s in zip(shapes, sets)]
    outs = [torch.full((bm.n_pairs(n),), -1, dtype=torch.int32, device="cuda:0") for m, n in shapes]
    torch.cuda.synchronize()
    batch = bm.Batch(ctx, idx, outs)
    batch.run()
    ctx.synchronize()
    batch.close()
    for shape, s, o in zip(shapes, sets, outs):
        assert np.array_equal(o.cpu().numpy().view(np.uint32), oracle.all_pairs(*s)), shape


@pytest.mark.parametrize("route", ["0", "1", None])
@pytest.mark.parametrize("prune", [0, 600])
def test_server_either_route(ctx, monkeypatch, route, prune):
    if route is not None:
        monkeypatch.setenv("BM_BITMAP_ROUTE", route)
    m, n = 30_000, 300
    rng = np.random.default_rng(11)
    off, tids = datagen.sets_from_probs(m, rng.uniform(0.001, 0.1, n), seed=12)
    items = np.flatnonzero(np.diff(off) >= prune)
    idx = bm.Index.from_sets(ctx, m, off, tids, max_loop=2, min_support=prune)
    srv = bm.Server(idx, streams=2, memory_budget=8 << 20, max_batch=5)
    queries = [rng.choice(items, size=k, replace=False).astype(np.uint32) for k in (2, 64, 65, 200, 3, 130, 17, 200, 90)]
    ids = [srv.submit(q) for q in queries]
    for q, i in zip(queries, ids):
        got, info = srv.wait(i, timeout_s=60.0)
        assert np.array_equal(got, oracle.subset_pairs(off, tids, q))
    srv.close()


@pytest.mark.parametrize("route", ["0", "1", None])
@pytest.mark.parametrize("m,n,count", [(700, 3, 1), (5_000, 40, 9880), (200_000, 30, 15), (40_000, 60, 777)])
def test_triples_either_route(ctx, monkeypatch, route, m, n, count):
    if route is not None:
        monkeypatch.setenv("BM_BITMAP_ROUTE", route)
    rng = np.random.default_rng(m + count)
    off, tids = datagen.sets_from_probs(m, rng.uniform(0.05, 0.9, n), seed=m)
    every = np.array([(a, b, c) for a in range(n) for b in range(a + 1, n) for c in range(b + 1, n)], np.uint32)
    pick = every if count == len(every) else rng.permuted(every[rng.integers(0, len(every), count)], axis=1)
    idx = bm.Index.from_sets(ctx, m, off, tids, order=3, max_loop=2)
    want = oracle.triples(off, tids, pick)
    for rep in range(2):
        assert np.array_equal(idx.triple_supports(pick, np.full(count, 3, np.uint32)), want)
    out = torch.full((count,), -1, dtype=torch.int32, device="cuda:0")
    dev = torch.from_numpy(pick.view(np.int32)).to("cuda:0")
    torch.cuda.synchronize()
    idx.triple_supports(dev, out)
    ctx.synchronize()
    assert np.array_equal(out.cpu().numpy().view(np.uint32), want)


@pytest.mark.parametrize("ingest", ["0", "1", None])       # radix sort, bit rows, by time
@pytest.mark.parametrize("m,n,deg", [
    (1, 3, 2), (255, 40, 3), (256, 41, 9), (257, 200, 0.3), (5_000, 1300, 20), (140_000, 37, 6), (9_000, 2400, 50),
    (300_000, 300, 10), (2_000, 5_000, 30),                  # the last: too many items for the bit rows' block
])
def test_transactions_either_ingest(ctx, monkeypatch, ingest, m, n, deg):
    """Transactions in any order with repeats and empty ones; the tidlists through both ways of counting."""
    if ingest is not None:
        monkeypatch.setenv("BM_BIT_INGEST", ingest)
    rng = np.random.default_rng(m + n)
    sizes = rng.poisson(deg, m) * (rng.random(m) < 0.9)
    sizes[-1] = 2
    hot = np.minimum((rng.random(int(sizes.sum())) ** 4 * n).astype(np.uint32), n - 1)   # a few items in most rows
    rows = np.zeros(m + 1, np.uint64)
    np.cumsum(sizes, out=rows[1:])
    off, tids = oracle.transpose(m, rows, hot, n)
    want = oracle.all_pairs(off, tids)
    dev = [torch.from_numpy(a).to("cuda:0") for a in (rows.view(np.int64), hot.view(np.int32))]
    torch.cuda.synchronize()
    for r, it in ((rows, hot), dev):
        idx = bm.Index.from_transactions(ctx, n, r, it)
        assert idx.stats()["nnz"] == tids.size
        for route in ("0", "1"):
            monkeypatch.setenv("BM_BITMAP_ROUTE", route)
            assert np.array_equal(idx.all_pair_supports(), want)
    bad = hot.copy()
    bad[bad.size // 2] = n
    with pytest.raises(bm.BatmapError) as e:
        bm.Index.from_transactions(ctx, n, rows, bad)
    assert e.value.status == bm.BM_ERANGE


def test_rows_kept_by_the_build(monkeypatch):
    """An index built through its bit rows has no slot plan: a capture before any eager call, and the
    allocation-free call, count from the rows."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    monkeypatch.setenv("BM_BIT_INGEST", "1")
    stream = torch.cuda.Stream()
    c = bm.Context(0, stream)
    for m, n, p in ((40_000, 300, 0.05), (3_000, 900, 0.1)):
        off, tids = datagen.bernoulli_sets(m, n, p, seed=n)
        rows, items = datagen.sets_to_transactions(m, off, tids)
        want = oracle.all_pairs(off, tids)
        idx = bm.Index.from_transactions(c, n, rows, items)
        out = torch.zeros(want.size, dtype=torch.int32, device="cuda:0")
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream, capture_error_mode="thread_local"):
            idx.all_pair_supports(out)
        for rep in range(3):
            out.fill_(-1)
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            assert np.array_equal(out.cpu().numpy().view(np.uint32), want)
            assert np.array_equal(idx.all_pair_supports(), want)
        sigma = int(np.median(want)) + 1
        fp = torch.zeros(3 * want.size, dtype=torch.int32, device="cuda:0")
        torch.cuda.synchronize()
        for route in (None, "0", "1"):
            if route:
                monkeypatch.setenv("BM_BITMAP_ROUTE", route)
            k = idx.frequent_pairs_noalloc(sigma, fp)
            c.synchronize()
            got = fp.cpu().numpy().view(np.uint32)[:3 * k].reshape(k, 3)
            assert np.array_equal(got, oracle.frequent_pairs(off, tids, sigma))
        monkeypatch.delenv("BM_BITMAP_ROUTE")
        del g
    c.close()
