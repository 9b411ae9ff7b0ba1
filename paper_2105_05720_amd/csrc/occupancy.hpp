// How many workgroups of the fused Adam kernels share a compute unit on shards bound by HBM, set through LDS that the launch
// asks for and nobody uses.  No HIP in here: the host can run it as well.
#pragma once

#include <stdint.h>

#include "cache_rules.hpp"

namespace ccf {

// Chunks of 1024 elements of a shard that does not fit the Infinity Cache (step's buffers of kResidentMaxBytes and more, the fused
// Adam step from kPlainLoadsMaxBytes on, see fused_policies) are bound by HBM, and what the addresses in flight look like decides: every XCD takes runs of 32 chunks (piece_in_runs), and the
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

// From kSmallShardElems elements on a plan's chunks are large and the ordered schedule takes over (up to eight fp32 slices), but the
// fused Adam step on one tensor for which nothing else was asked stays with single-wave pieces where they are the faster ones.
// One plan, the same buffers, large chunks and pieces in turn, us, medians of six (one shard by itself, then two in turn; where the
// arrays lie moves either side by up to 5 %):
//   fp16, R = 1       67 M elements 313 / 305, 318 / 295; 130 M 592 / 593, 600 / 577; 150 M 712 / 698, 689 / 667; but 201 M 904 / 931, 908 / 930
//   R = 2             67 M 330 / 313, 335 / 315; 130 M 644 / 617, 633 / 619; 201 M 981 / 952, 982 / 959
//   R = 4             67 M 372 / 354, 377 / 361; 130 M 721 / 720, 720 / 692; 201 M 1117 / 1091, 1140 / 1094
//   R = 8             67 M 451 / 442, 457 / 452; 130 M 871 / 863, 880 / 855; 201 M 1347 / 1325, 1351 / 1348
//   R = 10            67 M 498 / 483, 496 / 486; 130 M 964 / 952, 962 / 950; 201 M 1457 / 1457, 1466 / 1478
//   R = 12, 14, 16    level: 101 M 806 / 813, 875 / 889, 928 / 946; 201 M 1587 / 1611, 1736 / 1743, 1824 / 1878
//   fp32, R = 1 to 3  67 M 338 / 329, 373 / 353, 433 / 396; 130 M 636 / 624, 718 / 704, 850 / 779; 201 M 988 / 992, 1118 / 1074, 1302 / 1198
//   R = 4             67 M 461 / 430; 201 M 1425 / 1308; 400 M 2716 / 2597; 800 M 5721 / 5163
//   R = 8             67 M 646 / 627; 201 M 1961 / 1856; 400 M 4071 / 3774; 800 M 7797 / 7663
//   R = 12, 16        67 M 852 / 829, 1049 / 1030; 201 M 2596 / 2476, 3157 / 3079; 800 M 9726 / 9663, 12246 / 12127
// With fp16 slices and at least 260 M elements the ordered schedule is ahead (R = 1 1133 / 1181, R = 16 2474 / 2521; 500 M R = 1 2146 / 2244,
// R = 8 3285 / 3314).  With four and more fp32 slices, of which a compute unit's two chunks in flight are as much as it holds, the pieces
// were ahead at every size up to the 800 M elements measured, and the rule goes on beyond.
constexpr uint64_t kSmallShardElems = 64u << 20, kFlatNarrowMaxElems = 144u << 20, kFlatWideMaxElems = 192u << 20;
constexpr int kFlatMaxF16Slices = 10, kFlatAlwaysF32Slices = 4;
inline bool flat_beyond_small(uint64_t numel, int R, bool grad_f32)
{
    if (numel < kSmallShardElems || numel > kFlatMaxElems) return false;
    if (grad_f32) return numel < kFlatWideMaxElems || R >= kFlatAlwaysF32Slices;
    return R <= kFlatMaxF16Slices && numel < (R == 1 ? kFlatNarrowMaxElems : kFlatWideMaxElems);
}

// The fused LAMB step keeps its chunks of 1024 elements, one workgroup each, somewhat beyond: its first sweep gives the second m' and v' through
// the Infinity Cache (see cache_policies), which the ordered schedule's non-temporal stores do not, and the less of them fits the less
// that is worth.  More slices leave less room for them, and what a copy or a backward pass has left there takes its share.  If nothing was
// asked; us, ordered / this: one shard by itself, behind a 2 GiB copy, with the slices written just before, three shards in turn:
//   list, R = 1      67 M 454.9 / 414.3, 467.3 / 434.4, 462.5 / 427.7, 458.4 / 414.1   92 M 609.6 / 583.2, 621.9 / 603.0, 617.0 / 597.1, 616.3 / 580.2
//         R = 2      67 M 475.6 / 442.5, 487.1 / 462.5, 485.9 / 458.3, 474.9 / 437.1   92 M 632.7 / 614.2, 645.3 / 631.4, 645.7 / 634.3, 638.6 / 609.3
//         R = 4      74 M 570.7 / 537.3, 576.9 / 561.8, 575.4 / 558.9, 562.1 / 524.0   84 M 633.7 / 612.0, 642.4 / 634.2, 642.5 / 631.2, 634.5 / 609.8
//                    but 87 M 642.6 / 631.5, 652.9 / 662.1, 649.8 / 651.2, 643.4 / 622.8
//         R = 7      74 M 635.7 / 612.9, 645.2 / 635.5, 644.7 / 643.6, 632.1 / 601.4   84 M 720.0 / 698.1, 729.2 / 726.9, 728.3 / 727.2, 717.2 / 692.6
//         R = 8, 16  67 M 599.9 / 580.9, 609.8 / 613.7, 604.4 / 608.9, 600.9 / 575.7   67 M 787.7 / 782.0, 783.3 / 817.1, 778.0 / 820.0, 774.7 / 774.5
//         fp32 R = 3 74 M 624.5 / 591.2, 631.9 / 611.8, 632.3 / 628.4, 620.8 / 583.8; R = 4 74 M 665.7 / 637.7, 668.2 / 669.0, 663.2 / 681.6, 662.5 / 631.4
//   tensor, R = 1    75 M 506.2 / 483.8, 512.8 / 507.8, 509.0 / 491.3, 503.9 / 480.1   83 M 557.5 / 547.1, 564.1 / 568.8, 558.7 / 556.6, 558.2 / 547.5
//         R = 2      75 M 521.0 / 507.6, 529.7 / 529.4, 525.4 / 522.3, 520.4 / 503.7   91 M 630.6 / 627.2, 637.4 / 646.8, 636.6 / 640.3, 627.4 / 618.4
//         R = 4      71 M 538.7 / 529.1, 544.6 / 562.0, 541.0 / 545.6, 540.9 / 522.8
constexpr uint64_t kLambFewSlicesMaxElems = 88u << 20, kLambSomeSlicesMaxElems = 80u << 20, kLambOneTensorMaxElems = 72u << 20;
constexpr int kLambFewSliceBytes = 4, kLambSomeSliceBytes = 14;
inline bool lamb_keeps_small_chunks(uint64_t numel, int R, bool grad_f32, bool one_tensor)
{
    const int bytes = (grad_f32 ? 4 : 2) * R;
    if (bytes <= kLambFewSliceBytes) return numel < (one_tensor ? kLambOneTensorMaxElems : kLambFewSlicesMaxElems);
    return !one_tensor && bytes <= kLambSomeSliceBytes && numel < kLambSomeSlicesMaxElems;
}

// A list of tensors goes in such pieces as well, with the same reservations (flat_lds), where its step stores too much to write through:
// below kSmallShardElems instead of 128-thread workgroups, beyond instead of the ordered schedule, if nothing else was asked.
// us, without / with pieces, three shards in turn, then one by itself:
//   BERT-Large list   22 M, R = 1 103.5 / 101.7, 102.7 / 100.5; R = 4 126.4 / 123.9, 124.8 / 122.1; R = 8 157.0 / 155.8, 154.2 / 150.3; R = 12 185.5 / 186.2, 182.5 /
//                     183.5; 26 M, fp32 R = 1 128.3 / 125.3, 127 / 122.5; R = 4 181 / 174.5, 179 / 172; 34 M, R = 8 232.5 / 226.8, 230.9 / 223.5; R = 16 326.8 / 326.7,
//                     317.4 / 326.0; 42 M, R = 1 194.3 / 189, 194.8 / 186.5; R = 8 295 / 284.5, 290.8 / 279; R = 10 321 / 312, 312 / 311; 56 M, fp32 R = 8 567 / 521, 561 / 516
//   GPT-2 list        43 M, R = 2 214.5 / 209, 215 / 207; 56 M, R = 4 313.6 / 302, 313.6 / 299.7; R = 16 540 / 537, 530 / 540; 43 M, fp32 R = 16 674.5 / 674, 659 / 663
//   beyond, ordered / pieces: BERT-Large list 67 M, R = 1 321 / 300, 311 / 304; R = 8 480 / 456, 464 / 453; 84 M, R = 1 383 / 376, 383 / 374.5; R = 4 476 / 460, 462 /
//                     448.5; R = 8 576 / 571, 561.5 / 564; R = 10 629 / 629.5, 615 / 631; 111 M, R = 1 508 / 485, 500 / 494; R = 8 760 / 748, 739 / 748; but 168 M,
//                     R = 4 925 / 908, 908 / 901, 208 M, R = 8 1385 / 1394, 1367 / 1405, and 336 M, R = 8 2228 / 2248
//   ... fp32          67 M, R = 2 395 / 371, 380 / 367; 111 M, R = 4 772 / 745, 783 / 740; 168 M, R = 4 1219 / 1142, 1169 / 1121; 195 M, R = 8 1980 / 1875, 1908 / 1821;
//                     208 M, R = 4 1479 / 1385, 1445 / 1411; 336 M, R = 8 3460 / 3304, 3287 / 3368; 111 M, R = 16 1699 / 1699, 1732 / 1736
// It holds behind other work as well; one shard by itself, behind a 2 GiB copy, with the slices written just before, three in turn, without / with:
//   BERT-Large list   22 M, R = 8 154.6 / 150.7, 156.8 / 153.0, 152.5 / 151.6, 154.9 / 153.3; R = 10 168.9 / 170.4, 170.8 / 168.5, 168.3 / 163.9, 167.5 / 169.5; 42 M, R = 1
//                     193.0 / 188.5, 195.4 / 190.5, 192.5 / 190.0, 191.4 / 187.1; R = 8 292.1 / 278.6, 293.7 / 282.1, 288.9 / 281.6, 290.7 / 278.6; fp32 R = 8 418.3 /
//                     394.2, 416.8 / 397.8, 406.1 / 385.5, 410.6 / 391.7; 67 M, R = 1 320.3 / 309.2, 318.7 / 308.9, 314.9 / 302.8, 315.9 / 301.1; R = 8 470.9 / 459.8,
//                     472.6 / 455.4, 471.7 / 456.4, 468.1 / 450.8; 84 M, R = 1 383.1 / 387.0, 386.5 / 389.4, 381.7 / 385.9, 389.0 / 378.5; 112 M, R = 8 748.9 / 750.7,
//                     752.2 / 748.5, 748.9 / 745.7, 759.0 / 745.0; fp32 R = 4 778.5 / 778.8, 779.0 / 752.8, 775.9 / 750.7, 774.1 / 754.5
// While the stores are written through it depends on who steps: 10.5 M, R = 4 65.7 / 63.8 with three in turn, 54.8 / 57.3 by itself.
// Short chunks leave pieces without elements, so no more than one chunk in eight may be missing from the table.
constexpr uint64_t kListPiecesMaxElems = 128u << 20, kListPiecesMaxF32Elems = 256u << 20;
constexpr int kListPiecesMaxF16Slices = 10, kListBeyondMaxF16Slices = 8, kListPiecesMaxF32Slices = 8;
constexpr bool pieces_take(int R, bool grad_f32) { return R <= (grad_f32 ? kListPiecesMaxF32Slices : kListPiecesMaxF16Slices); }
// nothing_asked: beyond kSmallShardElems whoever asks for chunks of 1024 elements gets a workgroup for each.
inline bool list_in_pieces(uint64_t numel, uint64_t chunks, int R, bool grad_f32, bool nothing_asked)
{
    if (!pieces_take(R, grad_f32) || numel * kAdamStoreBytes < kWriteThroughMaxStoreBytes || chunks * 1024u > numel + numel / 8) return false;
    if (numel < kSmallShardElems) return true;
    if (!nothing_asked) return false;
    return grad_f32 ? numel < kListPiecesMaxF32Elems : R <= kListBeyondMaxF16Slices && numel < kListPiecesMaxElems;
}

}  // namespace ccf
