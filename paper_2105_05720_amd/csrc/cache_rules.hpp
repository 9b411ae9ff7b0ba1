// Which cache policy each kernel family of a plan uses.  No HIP in here: the host can run it as well.
#pragma once

#include <stdint.h>

#include "ccfused.h"

namespace ccf {

// AUTO cache policy: plain loads and write-through stores instead of non-temporal accesses while the step's buffers (R
// gradient slices, both copies of w, m, v and of the fp16 weights) total between these bounds, i.e. fit the 256 MB
// Infinity Cache.  Size sweep at R = 8, us per step: 6.2 against 7.9 at 2^20 elements (44 MB), 14.9 against 15.8 at 2^21
// (88 MB), 27.6 against 29.6 at 2^22 (176 MB), but 68.1 against 60.2 at 2^23 (352 MB).  Below 2^17 elements the
// non-temporal accesses are the faster ones by 1-6 % (LAMB at 2^14: 7.7 against 8.0 us), hence the lower bound.
constexpr uint64_t kResidentMinBytes = 4ull << 20, kResidentMaxBytes = 200ull << 20;
// ... and from there on non-temporal loads with write-through stores while one Adam launch stores less than this (see
// WriteThrough): what it writes then about fits the Infinity Cache.  One tensor at R = 8: 141 against 147 us at 20 Mi
// elements, 160 against 157 us at 22 Mi.  It holds for a list as well.  BERT-Large list cut into slices, written through /
// non-temporal, us, for 8.4 M, 14 M and 18.7 M elements at R = 8: back to back 54.1 / 60.1, 87.0 / 96.7, 114.6 / 129; behind
// sixteen matrix products and pointwise passes, as a backward pass is, 59.0 / 63.5, 93.0 / 101, 120 / 132; with the
// gradient slices written after those 57.9 / 59.7, 90.3 / 94.8, 119 / 130; behind a 2 GiB copy 60.0 / 63.6, 94.8 / 101, 124 / 132.
// Only a program that steps several such shards right behind each other has it the other way (three in turn: 63.3 / 61.7, 104 /
// 98.9, 136 / 130).
constexpr uint64_t kWriteThroughMaxStoreBytes = 288ull << 20;
inline uint64_t step_footprint(uint64_t numel, int R, bool grad_f32) { return numel * ((grad_f32 ? 4u : 2u) * (uint64_t)R + 12u + 14u); }
constexpr uint64_t kAdamStoreBytes = 14, kLambStoreBytes = 8;      // per element: w', m', v', w16 / m', v' (LAMB's first sweep)
inline int32_t auto_cache_policy(uint64_t footprint, uint64_t stored)
{
    if (footprint < kResidentMinBytes) return CC_CACHE_STREAMING;
    if (footprint < kResidentMaxBytes) return CC_CACHE_RESIDENT;
    return stored < kWriteThroughMaxStoreBytes ? CC_CACHE_WRITE_THROUGH : CC_CACHE_STREAMING;
}
// LAMB goes by the 8 bytes per element that its first sweep stores, up to 36 Mi elements.  Beyond that its two sweeps want
// different stores: written through in the first, whose m' and v' the second reads again, non-temporal in the second, whose
// output nobody reads before the next step.  BERT-Large list in slices, R = 8, 42 M elements, non-temporal in both / write-through and
// non-temporal / write-through in both, us: back to back 370 / 349 / 353, behind matrix products and pointwise passes 375 / 360 /
// 353, three shards in turn 372 / 350 / 376.  Below, write-through in both is the better one wherever a program steps one shard
// (write-through and non-temporal / write-through in both, back to back, behind products, with the gradient slices written after
// those, behind a copy: 121.6 / 117.4, 127.1 / 126.7, 119.7 / 120.1, 132.5 / 129.7 at 14 M, 231.0 / 225.4, 238.8 / 237.3, 241.2 /
// 231.5, 251.6 / 246.2 at 28 M), if not with three in turn (122.3 / 124.6 and 234.5 / 250.0).  At 56 to 60 M elements the pair is 3 to
// 5 % ahead back to back and, with eight and more slices that were written just before, 0 to 3 % behind non-temporal in both.
// The unfused pipeline's update reads in its second sweep what the first one wrote and hands its own output to the cast, so both
// are written through: non-temporal in both / this, 42 M elements, R = 8 back to back 453 / 423, behind a copy 457 / 439; R = 1 363 / 337
// and 370 / 352; 56 M, R = 8 606 / 569 and 611 / 591; one tensor of 60 M, R = 4 581 / 535 and 578 / 548.

// What a plan's small-chunk kernels use, by kernel family (cc_cache_policy values).
struct CachePolicies {
    int32_t adam = CC_CACHE_STREAMING;          // the fused Adam step (what cc_plan_layout reports) and the unfused pipelines: reduce, Adam from the sum, cast
    int32_t lamb1 = CC_CACHE_STREAMING;         // fused LAMB's first sweep, and both behind the unfused pipeline's reduce
    int32_t lamb = CC_CACHE_STREAMING;          // fused LAMB's second sweep
};
// one_sweep: the chunks are one sweep of a workgroup (1024 elements).  LAMB's pair holds for those only: with 2048-element
// chunks, which a caller has to ask for, both sweeps keep the same.
inline CachePolicies cache_policies(int32_t asked, uint64_t numel, int R, bool grad_f32, bool one_sweep)
{
    if (asked != CC_CACHE_AUTO) return CachePolicies{asked, asked, asked};
    const uint64_t footprint = step_footprint(numel, R, grad_f32);
    CachePolicies c;
    c.adam = auto_cache_policy(footprint, numel * kAdamStoreBytes);
    c.lamb = auto_cache_policy(footprint, numel * kLambStoreBytes);
    c.lamb1 = footprint < kResidentMaxBytes || !one_sweep ? c.lamb : CC_CACHE_WRITE_THROUGH;
    return c;
}

}  // namespace ccf
