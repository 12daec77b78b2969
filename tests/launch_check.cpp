// The sizes of launches as the host computes them, built with plan.cpp (no GPU).
#include <cstdint>
#include <vector>

#include "../paper_1102_1003_amd/csrc/plan.h"

// Work-items of the launch that counts `count` triples; *covered: whether its runs
// and segments take in every triple and every word of a row.
extern "C" uint64_t triple_bits_items(uint64_t count, uint32_t m, uint32_t n_cu, int *covered)
{
    const uint64_t words = bm::bit_row_words(m);
    const bm::TripleBitsPlan p = bm::plan_triple_bits(count, words, n_cu);
    *covered = p.n_runs * bm::kTripleRun >= count && p.n_runs > 0 && p.n_work % p.n_runs == 0 &&
               p.n_work / p.n_runs * p.seg >= words && p.seg % 256 == 0 && p.blocks > 0;
    return (uint64_t)p.blocks * bm::kTripleThreads;
}

// Work-items of the largest launch that adds the parts of na x nb counts; *covered:
// whether the launches follow one another over all of them.
extern "C" uint64_t gram_reduce_items(uint32_t na, uint32_t nb, int tri, uint32_t m, uint32_t n_cu, int pinned,
                                      int *covered)
{
    const bm::GramPlan p = bm::plan_gram(na, nb, tri != 0, bm::bit_row_words(m), n_cu, pinned);
    const uint32_t fold = bm::gram_reduce_fold(p, 64);
    const uint64_t blocks = bm::gram_reduce_blocks(p, fold);
    uint64_t most = 0, first = 0;
    while (first < blocks) {
        const uint64_t n = bm::gram_reduce_launch(blocks, first);
        most = n > most ? n : most;
        first += bm::kReduceGrid;
        if (n != bm::kReduceGrid)
            break;
    }
    *covered = first >= blocks && blocks * 1024 == (uint64_t)p.tiles * p.tile * p.tile * fold && blocks < (1ull << 32) &&
               (uint64_t)p.groups * (p.tile == 256 ? 512 : 256) < (1ull << 32);
    return most * bm::kReduceThreads;
}

// Work-items of the launches that make bit rows from tidlists (rows), and from
// transactions and tidlists from them (ingest; 0: not done that way).
extern "C" uint64_t bit_rows_items(uint64_t rows, uint32_t m, int *fits)
{
    const uint64_t blocks = bm::bit_row_blocks(rows, bm::bit_row_words(m));
    *fits = bm::grid_fits(blocks, bm::kBitRowThreads);
    return blocks * bm::kBitRowThreads;
}
extern "C" uint64_t bit_ingest_items(uint32_t m, uint32_t n, uint32_t lds, uint32_t n_cu, int *whole)
{
    *whole = 1;
    if (!bm::bit_ingest_fits(m, n, lds, n_cu))
        return 0;
    const uint32_t tw = bm::txn_bits_words(m, n, lds, n_cu);
    const uint64_t blocks = bm::txn_bits_blocks(m, tw), last = (bm::bit_row_words(m) - 1) / tw;
    // every word of a row has a workgroup, and its first transaction 32 bits
    *whole = blocks > last && last * (32ull * tw) < (1ull << 32);
    const uint64_t rows = blocks * bm::kTxnBitsThreads, segs = bm::bit_ingest_segments(m, n) * 256;
    return rows > segs ? rows : segs;
}

// Expected time of the count by transactions: nnz incidences of independent sets of
// equal size, and `longs` transactions of d items.
extern "C" double txn_price(uint32_t n, uint32_t m, double p, uint32_t longs, uint32_t d)
{
    const double nnz = (double)n * m * p;
    bm::TxnWalk w;
    w.pairs = (uint64_t)(nnz * nnz / (2.0 * m) + longs * 0.5 * d * (d - 1.0));
    if (d > bm::kTxnLong && longs) {
        w.long_items = (uint64_t)longs * d;
        w.long_squares = w.long_items * d;
        w.longest = d;
    }
    return bm::txn_us(n, (uint64_t)nnz + (uint64_t)longs * d, (uint32_t)(m * p) + longs, w, 256);
}

// The cut without scratch: 0, or what is wrong with it.
extern "C" int gram_add_check(uint32_t na, uint32_t nb, int tri, uint32_t m, uint32_t n_cu, int pinned)
{
    const bm::GramPlan p = bm::plan_gram_add(na, nb, tri != 0, bm::bit_row_words(m), n_cu, pinned);
    const uint64_t U = (uint64_t)p.tiles * p.stages, W = p.groups;
    if (W == 0 || W > U || p.ws_floats || (pinned && p.tile != pinned))
        return 1;
    bool shared = false;
    for (uint64_t w = 0; w < W; w++) {
        const uint64_t u0 = U * w / W, u1 = U * (w + 1) / W;
        shared = shared || u0 % p.stages != 0 || u1 % p.stages != 0;
        // the longest part of a tile in the run
        if (u1 - u0 > bm::kGramMaxStages && p.stages > bm::kGramMaxStages)
            return 2;
    }
    return shared && !p.add ? 3 : 0;
}

// Expected times of counting all pairs among maps of these classes (widths and counts,
// narrowest first) by slots and from bit rows of m transactions.
extern "C" void route_prices(const uint32_t *r, const uint32_t *count, uint32_t n_cls, uint32_t planes, uint32_t m,
                             int corrections, double *slots, double *bits)
{
    std::vector<bm::Cls> cls;
    uint32_t maps = 0;
    for (uint32_t c = 0; c < n_cls; c++) {
        cls.push_back({r[c], maps, count[c]});
        maps += count[c];
    }
    const bm::CompareLoad l = bm::compare_load(cls, planes);
    *slots = 10 + (corrections ? 5 : 0) + l.wait_us + l.work_us;
    *bits = bm::plan_gram(maps, maps, true, bm::bit_row_words(m), 256).us;
}
