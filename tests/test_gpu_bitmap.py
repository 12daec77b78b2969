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
