// The order in which the workgroups of a grid take the pieces of a call.  No HIP in here: the host can run it as well.
#pragma once

#include <stdint.h>

#if defined(__HIP__)
#define CCF_ANYWHERE __host__ __device__ __forceinline__
#else
#define CCF_ANYWHERE inline
#endif

namespace ccf {

// Which piece workgroup `b` of a grid of `grid` takes when every XCD is to own runs of consecutive pieces.  The hardware
// deals workgroups to the eight XCDs in turn, so taking piece b scatters neighbouring pieces over all of them; here the
// workgroups of one XCD take 2^RUN_LOG2 consecutive ones (64 KiB of an fp16 array: 64 of the epilogue's pieces of 512
// elements, 32 of the optimizer kernels' small chunks of 1024), the next XCD the run behind it.  A round of eight runs
// covers the same pieces either way, and what is left of the grid behind the last full round is taken in order, so every
// piece is taken exactly once.  Pays once the grid is a few rounds deep; on one or two rounds it only costs the imbalance.
template <uint32_t RUN_LOG2 = 6>
CCF_ANYWHERE uint32_t piece_in_runs(uint32_t b, uint32_t grid)
{
    constexpr uint32_t kRoundLog2 = RUN_LOG2 + 3;
    const uint32_t round = b >> kRoundLog2, in = b & ((1u << kRoundLog2) - 1u);
    if (round >= grid >> kRoundLog2) return b;
    return (round << kRoundLog2) + ((in & 7u) << RUN_LOG2) + (in >> 3);
}

// A launch has less than 2^32 threads.  A call whose pieces would need more goes out as several launches of `most` elements
// and what is left: launch(first element, elements) for each, in order.
template <class Launch>
inline void in_launches(uint64_t numel, uint64_t most, Launch launch)
{
    for (uint64_t done = 0; done < numel; done += most) launch(done, numel - done < most ? numel - done : most);
}

}  // namespace ccf
