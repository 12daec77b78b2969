"""Captured calls count from what the index holds, and make nothing inside the capture; every replay against
the oracle's merge, with eager work and other builds on the context in between."""
import numpy as np
import pytest

import datagen
import oracle

torch = pytest.importorskip("torch")
bm = pytest.importorskip("paper_1102_1003_amd")

pytestmark = pytest.mark.gpu


@pytest.fixture()
def stream_ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    stream = torch.cuda.Stream()
    c = bm.Context(0, stream)
    yield stream, c
    c.close()


def replays(stream, c, call, out, want, between):
    """Captures call(out) and replays it, with between() before each replay."""
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream, capture_error_mode="thread_local"):
        call(out)
    for rep in range(3):
        between()
        out.fill_(-1)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy().view(np.uint32), want)
    del g


@pytest.mark.parametrize("route", [None, "0", "1", "2"])
def test_after_an_eager_call(stream_ctx, monkeypatch, route):
    """More items than a build plans for: the eager call leaves a plan, rows or grouped incidences."""
    stream, c = stream_ctx
    if route is not None:
        monkeypatch.setenv("BM_BITMAP_ROUTE", route)
    m, n = 200_000, 5_000
    off, tids = datagen.bernoulli_sets(m, n, 0.0005, seed=5)
    want = oracle.all_pairs(off, tids, threads=0)
    idx = bm.Index.from_sets(c, m, off, tids)
    out = torch.zeros(want.size, dtype=torch.int32, device="cuda:0")
    torch.cuda.synchronize()
    c.set_profiling(True)
    idx.all_pair_supports(out)
    assert (c.timings()["compare_slot_pairs"] > 0) == (route == "0")     # by time: the incidences
    c.set_profiling(False)
    assert np.array_equal(out.cpu().numpy().view(np.uint32), want)

    def between():
        o, t = datagen.bernoulli_sets(9_000, 4_500, 0.01, seed=6)
        other = bm.Index.from_sets(c, 9_000, o, t)
        other.all_pair_supports()
        other.close()
    replays(stream, c, idx.all_pair_supports, out, want, between)
    assert np.array_equal(idx.all_pair_supports(), want)


@pytest.mark.parametrize("route", [None, "0"])
def test_nothing_made_inside(stream_ctx, monkeypatch, route):
    """A capture before any eager call is refused where there is nothing to count from, and leaves no plan behind."""
    stream, c = stream_ctx
    if route is not None:
        monkeypatch.setenv("BM_BITMAP_ROUTE", route)
    m, n = 30_000, 4_200
    off, tids = datagen.bernoulli_sets(m, n, 0.001, seed=7)
    want = oracle.all_pairs(off, tids, threads=0)
    idx = bm.Index.from_sets(c, m, off, tids)
    out = torch.zeros(want.size, dtype=torch.int32, device="cuda:0")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream, capture_error_mode="thread_local"):
        with pytest.raises(bm.BatmapError) as e:
            idx.all_pair_supports(out)
        out.zero_()
    assert e.value.status == bm.BM_EINVAL
    del g
    for rep in range(2):
        assert np.array_equal(idx.all_pair_supports(), want)
    replays(stream, c, idx.all_pair_supports, out, want, lambda: None)


def test_plan_of_the_other_launch_form(stream_ctx, monkeypatch):
    """A plan made for one launch form still serves a capture after the form has changed."""
    stream, c = stream_ctx
    monkeypatch.setenv("BM_BITMAP_ROUTE", "0")
    m, n = 20_000, 400
    off, tids = datagen.bernoulli_sets(m, n, 0.02, seed=8)
    want = oracle.all_pairs(off, tids)
    idx = bm.Index.from_sets(c, m, off, tids)
    out = torch.zeros(want.size, dtype=torch.int32, device="cuda:0")
    torch.cuda.synchronize()
    c.set_launch_mode(True)
    replays(stream, c, idx.all_pair_supports, out, want, lambda: None)
    c.set_launch_mode(False)


@pytest.mark.parametrize("tile", [0, 64, 128, 256])
@pytest.mark.parametrize("m,n,p", [(500, 2, 0.5), (1_000_000, 70, 0.002), (20_000, 300, 0.05), (3_000, 1_100, 0.02),
                                   (2**24 + 600_000, 3, None)])
def test_product_without_scratch(stream_ctx, monkeypatch, tile, m, n, p):
    """The bitmap product captured: its graph shares no scratch with eager calls or other graphs."""
    stream, c = stream_ctx
    if tile:
        monkeypatch.setenv("BM_GRAM_TILE", str(tile))
    if p is None:                                        # full sets: a count that fp32 cannot hold
        off = np.arange(n + 1, dtype=np.uint64) * m
        tids, want = np.tile(np.arange(m, dtype=np.uint32), n), np.full(3, m, np.uint32)
    else:
        off, tids = datagen.bernoulli_sets(m, n, p, seed=n)
        want = oracle.all_pairs(off, tids)
    idx = bm.Index.from_sets(c, m, off, tids)
    out = torch.full((want.size,), -1, dtype=torch.int32, device="cuda:0")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream, capture_error_mode="thread_local"):
        with pytest.raises(bm.BatmapError) as e:         # no rows yet: none are made inside a capture
            idx.all_pair_supports_dense(out)
        out.zero_()
    assert e.value.status == bm.BM_EINVAL
    del g
    assert np.array_equal(idx.all_pair_supports_dense(), want)
    replays(stream, c, idx.all_pair_supports_dense, out, want,
            lambda: np.testing.assert_array_equal(idx.all_pair_supports_dense(), want))


def test_waiting_calls_are_refused_whole(stream_ctx):
    """Calls that wait for the device: refused under capture before they grow a buffer or queue anything, so
    the capture stays valid and later eager calls work on memory of their own."""
    stream, c = stream_ctx
    m, n = 20_000, 260
    off, tids = datagen.bernoulli_sets(m, n, 0.03, seed=11)
    rows, items = datagen.sets_to_transactions(m, off, tids)
    want = oracle.all_pairs(off, tids)
    idx, other = (bm.Index.from_sets(c, m, off, tids) for _ in range(2))
    triples = bm.Index.from_sets(c, m, off, tids, order=3)
    out = torch.full((want.size,), -1, dtype=torch.int32, device="cuda:0")
    pairs = torch.zeros(3 * want.size, dtype=torch.int32, device="cuda:0")
    rect = torch.zeros(n * n, dtype=torch.int32, device="cuda:0")
    q = np.arange(40, dtype=np.uint32)
    calls = [
        lambda: idx.frequent_pairs_into(5, pairs), lambda: idx.frequent_pairs_noalloc(5, pairs),
        lambda: idx.all_pair_supports(np.zeros(want.size, np.uint32)), lambda: idx.subset_pair_supports(q, out),
        lambda: bm.cross_pair_supports(idx, other, rect), lambda: bm.cross_pairs(idx, other, 3, pairs),
        lambda: triples.triple_supports([(0, 1, 2)]), lambda: bm.Index.from_sets(c, m, off, tids),
        lambda: bm.Index.from_transactions(c, n, rows, items), lambda: bm.Batch(c, [idx], [out]),
        lambda: bm.Server(idx, streams=1, memory_budget=1 << 20),
    ]
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream, capture_error_mode="thread_local"):
        for call in calls:
            with pytest.raises(bm.BatmapError) as e:
                call()
            assert e.value.status == bm.BM_EINVAL
        idx.all_pair_supports(out)                       # the capture is still good
    assert len(idx.frequent_pairs(5)) == int((want >= 5).sum())
    assert np.array_equal(idx.subset_pair_supports(q)[:bm.n_pairs(40)], oracle.subset_pairs(off, tids, q))
    assert np.array_equal(bm.cross_pair_supports(idx, other), oracle.cross(off, tids, off, tids).reshape(n, n))
    assert np.array_equal(triples.triple_supports([(0, 1, 2)]), oracle.triples(off, tids, np.array([[0, 1, 2]], np.uint32)))
    torch.cuda.synchronize()
    g.replay()
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy().view(np.uint32), want)
    del g


@pytest.mark.parametrize("m,n,p", [(10_000_000, 3, 0.005), (10_000_000, 12, 0.004), (100_000, 64, 0.05)])
def test_few_sets_go_over_to_slots(stream_ctx, m, n, p):
    """The rows that a build leaves count first and stay for other calls; a plan is made once calls have paid for it."""
    stream, c = stream_ctx
    off, tids = datagen.sets_from_probs(m, np.full(n, p), seed=7)
    want = oracle.all_pairs(off, tids, threads=0)
    idx = bm.Index.from_sets(c, m, off, tids)
    out = torch.zeros(want.size, dtype=torch.int32, device="cuda:0")
    torch.cuda.synchronize()
    slots = []
    for call in range(40):
        out.fill_(-1)
        torch.cuda.synchronize()
        c.set_profiling(True)
        idx.all_pair_supports(out)
        slots.append(c.timings()["compare_slot_pairs"] > 0)
        c.set_profiling(False)
        assert np.array_equal(out.cpu().numpy().view(np.uint32), want)
    assert not slots[0] and slots == sorted(slots)
    assert slots[-1] == (m == 10_000_000)
    replays(stream, c, idx.all_pair_supports, out, want, lambda: idx.frequent_pairs(1))
    idx.close()
