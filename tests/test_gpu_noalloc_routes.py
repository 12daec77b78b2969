"""bm_frequent_pairs_noalloc after calls that counted by transactions, and so left no plan of the compare."""
import numpy as np
import pytest

import datagen
import oracle

torch = pytest.importorskip("torch")
bm = pytest.importorskip("paper_1102_1003_amd")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,p", [
    (200_000, 5_000, 0.0005),      # the counts fill the scratch: no room for a plan beside them
    (60_000, 4_200, 0.001),
])
def test_after_counting_by_transactions(m, n, p):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    off, tids = datagen.bernoulli_sets(m, n, p, seed=n)
    ctx = bm.Context(0)
    idx = bm.Index.from_sets(ctx, m, off, tids)
    for rep in range(2):
        ctx.set_profiling(True)
        idx.all_pair_supports()
        assert ctx.timings()["compare_slot_pairs"] == 0
        ctx.set_profiling(False)
    every = oracle.all_pairs(off, tids, threads=0)
    i, j = np.triu_indices(n, 1)
    for sigma in (1, 2, 3):
        keep = every >= sigma
        want = np.stack([i[keep], j[keep], every[keep]], 1).astype(np.uint32)
        out = torch.zeros(3 * max(len(want), 1), dtype=torch.int32, device="cuda:0")
        torch.cuda.synchronize()
        assert idx.frequent_pairs_noalloc(sigma) == len(want)
        assert idx.frequent_pairs_noalloc(sigma, out) == len(want)
        ctx.synchronize()
        assert np.array_equal(out.cpu().numpy().view(np.uint32)[:3 * len(want)].reshape(-1, 3), want)
    ctx.close()


@pytest.mark.parametrize("route", [None, "0"])
def test_bound_above_every_set(monkeypatch, route):
    """No item, or one, reaches the bound: no pair; an index past the scratch is refused all the same."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if route is not None:
        monkeypatch.setenv("BM_BITMAP_ROUTE", route)
    off, tids = datagen.bernoulli_sets(20_000, 300, 0.02, seed=3)
    sizes = np.sort(np.diff(off))
    ctx = bm.Context(0)
    idx = bm.Index.from_sets(ctx, 20_000, off, tids)
    out = torch.full((300,), -1, dtype=torch.int32, device="cuda:0")
    torch.cuda.synchronize()
    for rep in range(2):
        for sigma in (int(sizes[-1]) + 1, int(sizes[-2]) + 1, 1 << 31):
            assert idx.frequent_pairs_noalloc(sigma, out) == 0 == idx.frequent_pairs_noalloc(sigma)
            assert len(idx.frequent_pairs(sigma)) == 0
        idx.all_pair_supports()
    assert (out == -1).all()
    big_off, big_tids = datagen.bernoulli_sets(1_000, 5_200, 0.01, seed=4)
    big = bm.Index.from_sets(ctx, 1_000, big_off, big_tids)
    with pytest.raises(bm.BatmapError) as e:
        big.frequent_pairs_noalloc(1 << 20)
    assert e.value.status == bm.BM_EINVAL
    ctx.close()
