// How many workgroups of the fused Adam kernels share a compute unit on shards bound by HBM, set through LDS that the launch
// asks for and nobody uses.  No HIP in here: the host can run it as well.
#pragma once

#include <stdint.h>

#include "cache_rules.hpp"

namespace ccf {

// Chunks of 1024 elements of a shard that does not fit the Infinity Cache (step's buffers of kResidentMaxBytes and more) are
// bound by HBM, and what the addresses in flight look like decides: every XCD takes runs of 32 chunks (piece_in_runs), and the
// fused Adam kernel asks for LDS that nobody uses, so that six of its 128-thread workgroups fit a compute unit instead of
// up to sixteen.  Together, us before / runs only / runs and six workgroups: 36.6 / 36.1 / 35.9 at 5.3 M elements, 82.0 /
// 81.1 / 80.3 at 11.2 M, 389.2 / 385.7 / 382.9 at 56 M.  LAMB's first sweep adds up its chunk behind a barrier and cannot
// spare the waves (42 M elements: 357 us for both phases, 382 us with ten waves per compute unit).
//
// Once a step stores too much to write through (kWriteThroughMaxStoreBytes), a list with more than 16 bytes of slices per element is left four workgroups per compute
// unit, and three with more than eight fp32 slices: with the addresses in scalar registers (see Descriptor) six of them hold
// more streams in flight than DRAM likes, where registers used to keep them at four.  BERT-Large list in slices, back to back and
// behind a 2 GiB copy, us before / six / four / three: 56 M elements, R = 12 455 / 469 / 456 / 490 and 458 / 473 / 458 / 510, R = 16 532 /
// 547 / 537 / 564 and 527 / 552 / 538 / 586, R = 9 401 / 409 / 403 / 444; 28 M, R = 16 266 / 272 / 266 / 283 and 265 / 276 / 269 / 299;
// twelve fp32 slices, 28 M 353 / 359 / 358 / 344 and 357 / 364 / 360 / 349, 56 M 720 / 723 / 716 / 689; eight, 28 M 285 / 273 / 269 /
// 268, 42 M with the slices written just before 431 / 414 / 403 / 408.  While the stores are written through, six is right or
// within 1 % (R = 12, 9.3 M elements 70.7 / 69.3 / 71.4 / 84.5).
constexpr unsigned kSpreadLds = 24000, kFourWorkgroupsLds = 40000, kThreeWorkgroupsLds = 54000;   // of 160 KiB
constexpr int kSixWorkgroupsMaxSliceBytes = 16, kFourWorkgroupsMaxF32Slices = 8;
inline unsigned list_lds(uint64_t numel, int R, bool grad_f32, bool non_temporal_stores)
{
    const bool large = non_temporal_stores && numel * kAdamStoreBytes >= kWriteThroughMaxStoreBytes;
    if (!large || (grad_f32 ? 4 : 2) * R <= kSixWorkgroupsMaxSliceBytes) return kSpreadLds;
    return grad_f32 && R > kFourWorkgroupsMaxF32Slices ? kThreeWorkgroupsLds : kFourWorkgroupsLds;
}

// One tensor that does not fit the Infinity Cache and stays below the ordered schedule: single-wave workgroups of one
// group per lane, in grid order, and so few of them per compute unit (LDS that nobody uses again) that the addresses in
// flight are a narrow window that moves through all streams.  Without a table a workgroup starts its loads at once, so a
// small one costs nothing.  How few depends on what a wave has in flight, 4 (bytes of a slice element x R + 12) per lane.
// The reservation is a straight line in that, close to what measured best (in parentheses): 10000 bytes at R = 1 (10000),
// 10800 at 2 (11600), 12400 at 4 (13312), 15600 at 8 and for four fp32 slices (16000), i.e. 16, 15, 13 and 10 workgroups per
// compute unit, one more than the best at R = 2 and 4; short launches want more waves (5 M elements, R = 8: 32.3 us with
// 10000, 33.7 with 16000).  So does a step on fp16 slices that writes through, where one shard is stepped by itself: at R = 8
// and 12 the line ends at 13600 bytes (12 workgroups).  us before / with 15600 / 13600, back to back, with the slices written just
// before, behind a 2 GiB copy: 7.6 M elements, R = 8 50.2 / 49.9 / 47.5, 51.7 / 52.8 / 50.3, 58.0 / 52.9 / 52.2; 11 M 70.8 / 70.6 / 67.2, 72.1 /
// 72.7 / 69.7, 79.9 / 72.2 / 71.7; 14 M 86.5 / 88.1 / 85.6, 88.8 / 90.1 / 87.7, 97.6 / 90.6 / 91.0; three shards in turn 81.6 / 73.8 / 74.4
// at 11 M; 12 M, R = 12 86.8 / 85.7 / 84.6.  R = 16 and fp32 slices are 0 to 2 % better off with 16000 (18 M, R = 16 behind a copy 178 /
// 172 / 174; four fp32 slices, 12 M 84.0 / 77.8 / 78.6).  us, one shard back to back, 128-thread workgroups per 1024 elements / this: R = 8 33 / 32 at 5 M
// elements, 176 / 166 at 25 M, 432 / 397 at 60 M; R = 1 141 / 133 at 30 M; R = 2 199 / 189 at 40 M; R = 16 88 / 82 at 10 M, 403 / 377 at
// 40 M, 577 / 566 at 60 M; four fp32 slices 74 / 74 at 12 M (behind a 2 GiB copy 83 / 78), 298 / 256 at 40 M.
constexpr int kFlatBlock = 64;
constexpr uint32_t kFlatPiece = kFlatBlock * 4;
constexpr uint64_t kFlatShortBytes = 300ull << 20, kFlatMaxElems = 1ull << 33;      // 2^31 threads: a launch has less than 2^32
constexpr unsigned kFlatMostLds = 16000, kFlatThroughMostLds = 13600;
constexpr int kFlatThroughMaxR = 12;
inline unsigned flat_lds(uint64_t numel, int R, bool grad_f32, bool non_temporal_stores)
{
    if (step_footprint(numel, R, grad_f32) < kFlatShortBytes) return 10000u;
    const unsigned lds = 4400u + 400u * ((grad_f32 ? 4u : 2u) * (unsigned)R + 12u);
    const unsigned most = !non_temporal_stores && !grad_f32 && R <= kFlatThroughMaxR ? kFlatThroughMostLds : kFlatMostLds;
    return lds < most ? lds : most;
}

// From kSmallShardElems elements on a plan's chunks are large and the ordered schedule takes over, but the fused Adam step on
// one tensor for which nothing else was asked stays with single-wave pieces while they are the faster ones (where the arrays lie
// moves either side by 1 to 2 %).  Two shards in turn,
// us, large chunks (ordered up to eight fp32 slices) / pieces: fp16 slices, 64 Mi elements R = 8 470 / 444, 128 Mi 914 / 875;
// 70 M elements R = 1 324 / 308, R = 2 347 / 338, R = 4 384 / 372, R = 16 667 / 651; 200 M R = 1 897 / 879, R = 2 957 / 953, R = 4 1092 /
// 1051, R = 8 1340 / 1327, R = 16 1891 / 1886 (150 M 1410 / 1417); but 260 M R = 1 1133 / 1181, R = 16 2474 / 2521 and 500 M R = 1 2146 /
// 2244, R = 4 2661 / 2676, R = 8 3285 / 3314.  With four and more fp32 slices, of which a compute unit's two chunks in flight are
// as much as it holds, at every size: R = 4 485 / 458 at 70 M, 1388 / 1318 at 200 M, 3467 / 3280 at 500 M; R = 8 694 / 665, 2018 / 1854,
// 4968 / 4557; R = 12 906 / 865 at 70 M; R = 16 1108 / 1070 and 3229 / 3117 at 200 M.
constexpr uint64_t kSmallShardElems = 64u << 20, kFlatF16MaxElems = 192u << 20;
constexpr int kFlatAlwaysF32Slices = 4;
inline bool flat_beyond_small(uint64_t numel, int R, bool grad_f32)
{
    if (numel < kSmallShardElems || numel > kFlatMaxElems) return false;
    return numel < kFlatF16MaxElems || (grad_f32 && R >= kFlatAlwaysF32Slices);
}

}  // namespace ccf
