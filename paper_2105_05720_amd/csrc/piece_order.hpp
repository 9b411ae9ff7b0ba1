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

// Whether the small chunks of a plan's step are taken in runs, by the bytes of the step's buffers: from 200 MiB on, where
// they do not stay in the Infinity Cache, in an Adam step; in a LAMB step from 240 MiB on, because both its sweeps are faster in
// table order while most of the state they share is still on chip.  LAMB, us before there were runs / with runs / in table order
// now: 5.3 M elements of the BERT-Large list, R = 8 (220 MiB) back to back 50.0 / 50.5 / 48.6, behind a 2 GiB copy 58.5 / 58.9 /
// 57.0; one tensor of 4 M elements, R = 16 (221 MiB) 53.2 / 51.7 / 50.0 and 62.2 / 59.8 / 59.2, eight fp32 slices (221 MiB) with
// the slices written just before 50.5 / 52.0 / 49.0; but 6 M elements of the list, R = 8 (252 MiB) 57.3 / 54.6 / 55.5 and 66.8 /
// 63.8 / 64.6.
constexpr uint64_t kAdamRunsMinBytes = 200ull << 20, kLambRunsMinBytes = 240ull << 20;
inline bool chunks_in_runs(uint64_t step_bytes, bool lamb) { return step_bytes >= (lamb ? kLambRunsMinBytes : kAdamRunsMinBytes); }

// A launch has less than 2^32 threads.  A call whose pieces would need more goes out as several launches of `most` elements
// and what is left: launch(first element, elements) for each, in order.
template <class Launch>
inline void in_launches(uint64_t numel, uint64_t most, Launch launch)
{
    for (uint64_t done = 0; done < numel; done += most) launch(done, numel - done < most ? numel - done : most);
}

}  // namespace ccf
