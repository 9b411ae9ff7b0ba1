// What cc_plan_autotune tries.  No HIP in here: the host can run it as well.
#pragma once

#include <stdint.h>

#include <vector>

#include "ccfused.h"

namespace ccf {

// One setting of a plan, as cc_plan_set_chunk_elems, cc_plan_set_schedule and cc_plan_set_cache_policy would make it.
struct Candidate {
    int32_t chunk_elems, schedule;
    uint32_t workgroups;
    int32_t cache;
};
struct TuningLayout {
    int32_t chunk_elems;
    int64_t chunks;
    bool small;         // 128-thread workgroups: the cache policies exist
    bool orders;        // the ordered schedule exists
};

// CC_SCHEDULE_PER_CHUNK with the current chunk size first, non-temporal (in single-wave pieces where those are the rule for such chunks): its
// time is what per_chunk_ms reports.  Small
// chunks are tried under every cache policy, and for LAMB under AUTO as well, which may give its two sweeps different ones
// (cache_policies), as no policy that is asked for does.  A plan for which nothing is chosen comes last: some of what it runs goes by
// that (single-wave pieces of large shards, few slices read plainly up to 144 MiB of buffers).  Without these two a tuned plan could be slower than an untuned one.
inline std::vector<Candidate> tuning_candidates(const std::vector<TuningLayout> &layouts, int32_t current, int32_t optimizer, uint32_t cus)
{
    std::vector<Candidate> c;
    auto per_chunk = [&](const TuningLayout &l) {
        c.push_back(Candidate{l.chunk_elems, CC_SCHEDULE_PER_CHUNK, 0u, CC_CACHE_STREAMING});
        if (!l.small) return;
        for (int32_t p : {CC_CACHE_RESIDENT, CC_CACHE_WRITE_THROUGH}) c.push_back(Candidate{l.chunk_elems, CC_SCHEDULE_PER_CHUNK, 0u, p});
        if (optimizer == 1) c.push_back(Candidate{l.chunk_elems, CC_SCHEDULE_PER_CHUNK, 0u, CC_CACHE_AUTO});
    };
    for (const TuningLayout &l : layouts)
        if (l.chunk_elems == current) per_chunk(l);
    for (const TuningLayout &l : layouts) {
        if (l.chunks == 0) continue;
        if (l.chunk_elems != current) per_chunk(l);
        if (l.orders)
            for (uint32_t w : {cus, cus > 1 ? cus / 2 : 1u, cus * 2}) c.push_back(Candidate{l.chunk_elems, CC_SCHEDULE_ORDERED, w, CC_CACHE_STREAMING});
    }
    c.push_back(Candidate{0, CC_SCHEDULE_AUTO, 0u, CC_CACHE_AUTO});
    return c;
}

}  // namespace ccf
