"""The launches that small builds and queries share: maps of one bucket chunk, block counts summed by the
threshold's writer, offsets checked by one workgroup.  Whole numbers: everything is compared exactly."""
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


@pytest.mark.parametrize("prune", [0, 100])
@pytest.mark.parametrize("m", [9_000, 600_000])        # with and without the table of hops
@pytest.mark.parametrize("widest", [1, 4095, 4096, 4097, 8192])
def test_bucket_chunks(ctx, monkeypatch, m, widest, prune):
    """Block-family maps below, at and past one chunk of 4,096 elements, empty ones among them."""
    monkeypatch.setenv("BM_BITMAP_ROUTE", "0")         # count from the maps themselves
    if widest < prune:
        pytest.skip("no map would be left")
    rng = np.random.default_rng(widest)
    sizes = [0, 1, min(widest, 700), widest, 0, max(widest - 1, 1), min(widest, 4096)]
    sets = [np.sort(rng.choice(m, s, replace=False)).astype(np.uint32) for s in sizes]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.uint64)
    tids = np.concatenate(sets).astype(np.uint32)
    idx = bm.Index.from_sets(ctx, m, off, tids, min_support=prune)
    keep = np.flatnonzero(np.array(sizes) >= prune)
    want = oracle.subset_pairs(off, tids, keep.astype(np.uint32))
    assert np.array_equal(idx.subset_pair_supports(keep.astype(np.uint32)), want)


@pytest.mark.parametrize("n", [2, 91, 92, 2896, 2897])  # one block of 4,096 pairs and two; 1,024 blocks and 1,025
def test_threshold_blocks(ctx, n):
    m = 300
    off, tids = datagen.bernoulli_sets(m, n, 0.2, seed=n)
    idx = bm.Index.from_sets(ctx, m, off, tids)
    sup = oracle.all_pairs(off, tids)
    sigma = int(np.quantile(sup, 0.9)) + 1
    i, j = np.triu_indices(n, 1)
    hit = sup >= sigma
    want = np.stack([i[hit], j[hit], sup[hit]], 1)
    total = len(want)
    out = torch.full((total + 2, 3), -1, dtype=torch.int32, device="cuda:0")
    torch.cuda.synchronize()
    assert idx.frequent_pairs_into(sigma, out) == total
    ctx.synchronize()
    got = out.cpu().numpy()
    assert np.array_equal(got[:total], want) and (got[total:] == -1).all()


@pytest.mark.parametrize("m", [1, 16_384, 16_385])
@pytest.mark.parametrize("fault", [None, "first", "last step"])
def test_device_offsets(ctx, m, fault):
    """Row offsets in device memory on both sides of the one-workgroup check: a start that is not 0, a decrease."""
    off = np.arange(m + 1, dtype=np.int64)
    if fault == "first":
        off[0] = 1
    if fault == "last step":
        if m == 1:
            pytest.skip("one step back from 0 is a count past 2^32")
        off[m] = off[m - 1] - 1
    d_off = torch.from_numpy(off).to("cuda:0")
    items = torch.zeros(max(m, 1), dtype=torch.int32, device="cuda:0")
    torch.cuda.synchronize()
    if fault:
        with pytest.raises(bm.BatmapError):
            bm.Index.from_transactions(ctx, 2, d_off, items)
    else:
        idx = bm.Index.from_transactions(ctx, 2, d_off, items)
        assert idx.all_pair_supports().tolist() == [0]
