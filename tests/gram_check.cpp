// Host checks of plan_gram, built with plan.cpp (no GPU).
#include <cstdint>
#include <cstdio>
#include <set>
#include <vector>

#include "../paper_1102_1003_amd/csrc/plan.h"

// Walks every group's run as the Gram kernel does: 0, or a message.  Each
// (tile, stage) is visited once, no run part passes the fp32 bound, each shared
// part has a place of its own inside ws, and gram_reduce_kernel's rule finds it.
static int check_plan(const bm::GramPlan &p, uint32_t na, uint32_t nb, uint32_t m, uint64_t max_ws, char *msg,
                      uint32_t len)
{
    const uint64_t U = (uint64_t)p.tiles * p.stages, W = p.groups;
    auto bad = [&](const char *what) {
        snprintf(msg, len, "%s: tile %d tiles %u stages %u groups %u", what, p.tile, p.tiles, p.stages, p.groups);
        return 1;
    };
    if ((uint64_t)p.tile_rows * p.tile < na || (uint64_t)p.tile_cols * p.tile < nb)
        return bad("counts left out");
    if ((uint64_t)p.stages * bm::kGramStage < m || W == 0 || W > U)
        return bad("bad cut");
    if (p.ws_floats > max_ws && p.stages <= bm::kGramMaxStages && max_ws == 0)
        return bad("scratch where none was to be used");
    if (p.ws_floats > max_ws && (uint64_t)p.stages * p.tiles <= bm::kGramMaxStages && max_ws >= 2ull * 256 * 256)
        return bad("more scratch than allowed");
    uint64_t seen = 0;
    std::set<uint64_t> places;
    for (uint64_t w = 0; w < W; w++) {
        const uint64_t u0 = U * w / W, u1 = U * (w + 1) / W;
        if (u0 != seen || u1 <= u0)
            return bad("runs do not follow one another");
        for (uint64_t u = u0; u < u1;) {
            const uint64_t t = u / p.stages, s0 = u % p.stages;
            const uint64_t steps = p.stages - s0 < u1 - u ? p.stages - s0 : u1 - u;
            if (steps > bm::kGramMaxStages)
                return bad("a part passes the fp32 bound");
            if (steps != p.stages) {
                const uint64_t place = 2 * w + (u != u0);
                if ((place + 1) * p.tile * p.tile > p.ws_floats || !places.insert(place).second)
                    return bad("a part without a place of its own");
                // the reduction's rule: the first group's place is its second when it came from another tile
                const bool first = u == t * p.stages;
                if (place != 2 * w + (first && u0 != t * p.stages))
                    return bad("the reduction would look elsewhere");
            }
            u += steps;
        }
        seen = u1;
    }
    return seen == U ? 0 : bad("stages left out");
}

extern "C" int gram_check(uint32_t na, uint32_t nb, int tri, uint32_t m, uint32_t n_cu, int pinned, uint64_t max_ws,
                          char *msg, uint32_t len)
{
    const bm::GramPlan p = bm::plan_gram(na, nb, tri != 0, bm::bit_row_words(m), n_cu, pinned, max_ws);
    return check_plan(p, na, nb, m, max_ws, msg, len);
}

// The families of a joint launch: each cut as above, the scratch enough for all
// of them, the workgroups no more than three a compute unit unless every family
// is down to the fewest it can have.
extern "C" int gram_set_check(const uint32_t *n, const uint32_t *m, uint32_t count, uint32_t n_cu, int pinned,
                              uint32_t *joint, uint32_t *groups, char *msg, uint32_t len)
{
    std::vector<bm::GramShape> shapes;
    for (uint32_t q = 0; q < count; q++)
        shapes.push_back({n[q], bm::bit_row_words(m[q])});
    const bm::GramSetPlan set = bm::plan_gram_set(shapes, n_cu, pinned);
    uint64_t ws = 0, w = 0;
    bool least = true;
    *joint = 0;
    for (uint32_t q = 0; q < count; q++) {
        const bm::GramPlan &p = set.plan[q];
        if (check_plan(p, n[q], n[q], m[q], UINT64_MAX, msg, len))
            return 1;
        if (!set.joint[q]) {
            if (p.ws_floats > set.ws_floats) {
                snprintf(msg, len, "a single family's scratch");
                return 1;
            }
            continue;
        }
        ++*joint;
        ws += p.ws_floats;
        w += p.groups;
        least = least && ((uint64_t)p.groups - 1) * bm::kGramMaxStages < (uint64_t)p.tiles * p.stages;
        if (p.tile != 64 && p.tile != 128) {
            snprintf(msg, len, "a joint tile of %d", p.tile);
            return 1;
        }
    }
    *groups = set.groups;
    if (ws > set.ws_floats || w != set.groups || (w > 3ull * n_cu && !least)) {
        snprintf(msg, len, "%llu groups, %llu floats of %llu", (unsigned long long)w, (unsigned long long)ws,
                 (unsigned long long)set.ws_floats);
        return 1;
    }
    return 0;
}
