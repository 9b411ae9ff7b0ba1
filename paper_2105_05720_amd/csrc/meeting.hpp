// When a fused LAMB step is a single launch whose workgroups wait for each other's sums (see LambMeeting), and for how long they
// wait.  No HIP in here: the host can run it as well.
#pragma once

#include <stdint.h>

namespace ccf {

constexpr uint32_t kMeetingChunks = 64, kMeetingMostChunks = 512, kMeetingGroups = 64, kGroupCopies = 8;

// Looks of a wave at the other workgroups' sums (0.5 to 1 us each) before it gives up, how many times as long the half of the
// workgroups wait that stays, how often a wave that waits looks whether some have left, and how long one that came after that stays.
constexpr uint32_t kMeetingPolls = 64, kMeetingPatience = 64, kMeetingGlance = 16, kMeetingLinger = 8;
// ... and what ends even the waits of those who know that everybody will publish: some seconds.  Only calls that overlap on one
// plan, which mix their arrivals and words, get there.
constexpr uint32_t kMeetingBound = 1u << 22;
// Half of any eight workgroups in a row, and of any that are 2^k apart: workgroups go to XCDs, shader engines and compute
// units in turn, and on each some have to make room.
constexpr bool meeting_stays(uint32_t workgroup)
{
    for (int k = 16; k; k >>= 1) workgroup ^= workgroup >> k;
    return (workgroup & 1u) != 0u;
}

// Waves per SIMD that the kernel's registers leave room for, hence workgroups (of two waves) per compute unit: twice that.
// Four slices of fp16 take 116 registers, seven 167, eight fp32 slices 128, twelve 162.
constexpr int lamb_meeting_waves(int R, bool grad_f32)
{
    return grad_f32 ? (R <= 8 ? 4 : R <= 12 ? 3 : 2) : (R <= 4 ? 4 : R <= 7 ? 3 : 2);
}

inline bool lamb_meets(int64_t chunks, uint32_t groups, int32_t cus, int R, bool grad_f32)
{
    return chunks > 0 && chunks <= (int64_t)kMeetingMostChunks && groups <= kMeetingGroups
           && 2 * chunks <= (int64_t)cus * lamb_meeting_waves(R, grad_f32);
}

// Whether cc_fused_lamb_step's first sweep adds up the chunks' sums group by group and the second the groups (see LambTally), instead of
// a launch between the two.  `most`: chunks of the largest tensor.  One tensor and lists, us per step with the launch / without:
//   chunks       606 R = 2   684 R = 8   879 R = 4   1075 R = 8   1447 R = 1   2442 R = 2   2442 R = 16   3907 R = 8   5470 R = 2   7945 R = 4
//               11.2 / 10.1 12.8 / 11.7 12.9 / 11.6 14.7 / 13.5  14.8 / 13.1  22.4 / 21.0  34.1 / 33.3   39.5 / 38.2  41.1 / 40.6  63.2 / 61.8
//   15.6 K, R = 2 110.1 / 107.7; 19.5 K, eight fp32 slices 238 / 235.5; 27.3 K, R = 1 180.2 / 178.2; but 39.1 K, R = 8 336.0 / 338.4 and 58.6 K, R = 2
//   399 / 400.7.  BERT-Large list in 14 slices, R = 4 181.5 / 181.0, in 40, R = 8 74.3 / 73.5; GPT-2 list in 60, R = 4 198.3 / 196.0.
// Where no tensor has more than kFoldNormsMaxChunks the second sweep adds up the chunks themselves: BERT-Large list in 203 slices, R = 8, 19.5 us that
// way, 20.6 with the tally.  Between 512 and 600 chunks the launch stays as well, though the tally would be ahead there too: one tensor of 514, 538, 567 and 598 chunks,
// R = 1 10.6 / 9.3, 11.4 / 9.5, 11.8 / 9.6 and 11.4 / 9.5, R = 8 11.0 / 9.9, 11.5 / 10.2, 11.8 / 10.3 and 11.6 / 10.3, R = 16 11.9 / 10.9, 12.4 / 11.3, 12.5 / 11.3 and 12.7 / 11.6.
constexpr uint32_t kFoldNormsMaxChunks = 512;
constexpr int64_t kTallyMinChunks = 600, kTallyMaxChunks = 32768;
inline bool lamb_tallies(int64_t chunks, uint32_t most) { return chunks >= kTallyMinChunks && chunks <= kTallyMaxChunks && most > kFoldNormsMaxChunks; }

// Whether the phase calls do without that launch: every tensor is one group, and few enough of them (the counts and
// groups take 176 bytes each).  us for the two calls with the launch / without, eager, then graph replay: one tensor of 1031 elements, R = 2
// 12.4 / 9.1, 7.1 / 6.4; 10007, R = 8 12.4 / 9.1, 8.3 / 7.3; 65000, R = 1 12.4 / 9.2, 8.7 / 8.0; BERT-Large list in 512 slices, R = 8 13.3 / 11.5, 13.0 / 11.5;
// 8.3B list in 450, R = 4 23.6 / 22.3, 23.0 / 21.5.  With tensors of several groups, which the first sweep would have to add up as well, the
// two take the same time: the trips to memory at its end cost what the launch did (BERT-Large list in 203 slices, R = 2 16.6 / 16.9).
constexpr uint32_t kOneGroupChunks = 64;
constexpr int64_t kOneGroupEachMaxChunks = 8192;
inline bool lamb_one_group_each(int64_t chunks, uint32_t most) { return chunks > 0 && chunks <= kOneGroupEachMaxChunks && most <= kOneGroupChunks; }

}  // namespace ccf
