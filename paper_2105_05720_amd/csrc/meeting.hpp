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

}  // namespace ccf
