// The sizes of launches as the host computes them, built with plan.cpp (no GPU).
#include <cstdint>

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
