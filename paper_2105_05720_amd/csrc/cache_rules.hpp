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
    int32_t adam = CC_CACHE_STREAMING;          // what cc_plan_layout reports: the unfused pipelines (reduce, Adam from the sum, cast) and the fused Adam step, but see fused_policies
    int32_t lamb1 = CC_CACHE_STREAMING;         // fused LAMB's first sweep, and both behind the unfused pipeline's reduce
    int32_t lamb = CC_CACHE_STREAMING;          // fused LAMB's second sweep
    bool slices_plain = false;                  // fused Adam reads the gradient slices with plain loads whatever `adam` says of the state
};
// one_sweep: the chunks are one sweep of a workgroup (1024 elements).  LAMB's pair holds for those only: with 2048-element
// chunks, which a caller has to ask for, both sweeps keep the same.
inline CachePolicies cache_policies(int32_t asked, uint64_t numel, int R, bool grad_f32, bool one_sweep)
{
    if (asked != CC_CACHE_AUTO) return CachePolicies{asked, asked, asked, false};
    const uint64_t footprint = step_footprint(numel, R, grad_f32);
    CachePolicies c;
    c.adam = auto_cache_policy(footprint, numel * kAdamStoreBytes);
    c.lamb = auto_cache_policy(footprint, numel * kLambStoreBytes);
    c.lamb1 = footprint < kResidentMaxBytes || !one_sweep ? c.lamb : CC_CACHE_WRITE_THROUGH;
    return c;
}

// What the fused steps' launches use where AUTO says RESIDENT.  A plain load that misses places its line in the Infinity Cache, and
// where that is full of lines that others wrote (a backward pass, other shards), one of those goes to HBM first.  With the step's
// buffers at this size and beyond, a step finds too little of what it reads on chip to make up for that: its loads are
// non-temporal from there on, but for the weights in LAMB's first sweep, which the second reads again.  That one's loads stay
// plain as long as the w, m' and v' that it reads still fit the eight L2s.
// us, plain loads / this (Adam: one tensor, which then runs in single-wave pieces, see kFlatPiece; its 63 and 76 MB are below the line):
//                              three shards in turn   one by itself   behind a 1 GiB fill   behind a copy, with the slices written
//   Adam R = 8,   63 MB            11.4 / 11.7         10.6 / 10.9        24.0 / 15.7            14.5 / 14.1
//                 76 MB            13.2 / 13.9         13.0 / 12.6        28.2 / 17.7            16.8 / 15.7
//                 84 MB            15.5 / 14.9         14.3 / 13.6        30.9 / 18.8            18.4 / 16.8
//                126 MB            26.4 / 20.7         19.2 / 19.8        43.1 / 25.7            23.3 / 22.8
//                176 MB            35.8 / 27.8         27.2 / 27.6        58.0 / 34.2            31.6 / 29.5
//        R = 1,   84 MB            16.2 / 15.9         14.1 / 16.0        26.8 / 19.1            19.0 / 17.9
//        R = 16, 174 MB            36.7 / 27.5         28.9 / 27.1        62.4 / 33.8            32.5 / 29.2
//        list, 110 MB              22.0 / 20.0         18.7 / 18.9        40.6 / 25.7            22.9 / 22.1
//   LAMB R = 8,   63 MB            18.8 / 19.1         17.4 / 17.5        31.8 / 24.6            22.3 / 21.6
//                 84 MB            23.2 / 22.4         21.7 / 20.9        39.0 / 29.3            26.3 / 24.9
//                126 MB            36.3 / 31.3         30.3 / 29.2        53.4 / 38.4            34.7 / 32.4
//                176 MB            48.9 / 40.7         39.8 / 39.0        69.8 / 48.9            43.9 / 41.9
//        R = 1,  140 MB            41.4 / 35.5         36.0 / 33.8        55.1 / 44.7            43.0 / 39.0
// (LAMB with all loads of the first sweep non-temporal: 24.4 at 84 MB, 34.3 at 126.  Second sweep with plain / non-temporal loads, three in
// turn: 22.4 / 23.0 at 24 MB of w, m' and v', 27.1 / 27.4 at 30, 31.1 / 31.3 at 36, 41.5 / 40.7 at 50, R = 1 38.2 / 35.5 at 60.)
// Adam on few slices lost by that where one shard is stepped by itself, whose arrays are on chip from step to step: the loads
// of the state find them there either way, those of the slices, which nobody writes in between, only if they are plain.  So up to 4 bytes of
// slices per element are read plainly up to kSlicesPlainMaxBytes.  us, plain loads / all non-temporal / this, in the first four situations and
// with the slices written just before (behind a copy):
//                              three in turn            one by itself         behind a fill         behind a copy         slices written
//   one tensor, R = 1,  86 MB  16.7 / 16.5 / 14.3       14.4 / 15.7 / 13.6    28.2 / 19.4 / 20.0    21.2 / 19.0 / 18.7    20.0 / 18.4 / 18.3
//                      117 MB  23.1 / 22.2 / 19.0       18.6 / 21.0 / 18.1    36.5 / 24.7 / 25.5    26.3 / 23.2 / 22.9    24.4 / 22.6 / 22.2
//                      147 MB  28.4 / 25.9 / 23.6       22.5 / 26.0 / 22.4    42.8 / 29.2 / 30.8    30.9 / 26.6 / 27.1    28.8 / 26.2 / 26.3
//             R = 2,  117 MB   22.9 / 21.5 / 19.1       18.9 / 20.3 / 17.7    36.6 / 25.1 / 26.8    27.1 / 22.7 / 23.4    24.3 / 22.7 / 22.4
//             fp32 R = 1, 117  23.3 / 20.7 / 19.4       18.6 / 19.7 / 18.1    37.4 / 24.7 / 27.4    27.5 / 22.7 / 23.2    23.5 / 22.4 / 22.2
//   list, R = 1,      136 MB   28.8 / 25.8 / 24.5       22.4 / 25.9 / 21.8    43.8 / 30.5 / 32.0    30.3 / 26.6 / 27.1    28.3 / 26.0 / 26.0
//         R = 2,      136 MB   29.4 / 24.5 / 24.1       22.2 / 24.6 / 21.9    44.9 / 30.5 / 34.0    31.6 / 26.8 / 27.5    27.3 / 26.2 / 26.4
// Beyond that line, and with more slices, what the cold ones cost is more: one tensor, R = 1, 204 MB 38.1 / 33.5 / 35.1, 30.7 / 35.2 / 30.3, 59.1 / 38.4 / 40.2,
// 40.3 / 34.8 / 34.8; R = 2, 204 MB 38.5 / 32.9 / 35.4, 31.1 / 34.2 / 30.2, 60.0 / 38.2 / 42.6, 41.8 / 34.5 / 34.5; R = 4, 117 MB 23.4 / 20.3 / 19.7, 19.0 / 19.3 /
// 18.4, 39.0 / 24.5 / 29.6, 28.5 / 22.7 / 24.0.  There one shard by itself stays the slower one (R = 1 up to 16 %, R = 2 10 %, R = 4 6 %, R = 8 4 %; lists of several hundred tensors, plain / all non-temporal
// by itself, three in turn, behind a copy, slices written: R = 4, 133 MB 21.6 / 22.9, 28.6 / 23.3, 32.6 / 26.3, 26.0 / 25.3; R = 16, 152 MB 24.3 / 25.8, 34.4 / 27.2, 42.3 / 32.5, 29.0 /
// 28.8), and every other situation the faster.
constexpr uint64_t kPlainLoadsMaxBytes = 80ull << 20, kL2Bytes = 32ull << 20, kLambReadAgainBytes = 12;
constexpr uint64_t kSlicesPlainMaxBytes = 144ull << 20;
constexpr bool slices_plain_for(int R, bool grad_f32) { return (grad_f32 ? 4 : 2) * R <= 4; }
constexpr int32_t kWeightsKept = 16;       // beside the cc_cache_policy values: see WeightsKept in kernels.hip.h
inline CachePolicies fused_policies(CachePolicies c, int32_t asked, uint64_t numel, int R, bool grad_f32, bool one_sweep)
{
    const uint64_t footprint = step_footprint(numel, R, grad_f32);
    if (asked != CC_CACHE_AUTO || !one_sweep || footprint < kPlainLoadsMaxBytes || footprint >= kResidentMaxBytes) return c;
    c.adam = CC_CACHE_WRITE_THROUGH;
    c.slices_plain = slices_plain_for(R, grad_f32) && footprint < kSlicesPlainMaxBytes;
    c.lamb1 = kWeightsKept;
    if (numel * kLambReadAgainBytes >= kL2Bytes) c.lamb = CC_CACHE_WRITE_THROUGH;
    return c;
}

}  // namespace ccf
