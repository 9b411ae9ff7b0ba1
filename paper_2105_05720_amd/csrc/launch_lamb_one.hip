// The small LAMB step in one launch (see LambMeeting).
#include "plan.hpp"

namespace ccf {

namespace {

template <bool GF32, bool GROUPED, class MEM>
void launch_lamb_one_r(const cc_plan *p, const StepScalars &s, int32_t *flag, hipStream_t st)
{
    const Layout &L = p->lamb_lay();
    const dim3 grid((unsigned)L.chunks), block(kSmallBlock);
    switch (p->R) {
#define CASE(r) case r: hipLaunchKernelGGL((lamb_one_launch_kernel<GradSlices<r, GF32, MEM>, GROUPED, kSmallBlock, lamb_meeting_waves(r, GF32)>), grid, block, 0, st, L.d_per_chunk, s, p->d_sums, p->d_meeting, flag, p->meeting_limit, L.groups); break;
        FOR_EACH_R(CASE)
#undef CASE
    }
}

// Up to 65536 elements every wave looks at every chunk's sums, beyond that at every group's.
template <bool GF32, class MEM>
void launch_lamb_one(const cc_plan *p, const StepScalars &s, int32_t *flag, hipStream_t st)
{
    if (p->lamb_lay().chunks > (int64_t)kMeetingChunks) launch_lamb_one_r<GF32, true, MEM>(p, s, flag, st);
    else launch_lamb_one_r<GF32, false, MEM>(p, s, flag, st);
}

// A shard this small has the same policy in both sweeps (see cache_policies).
template <bool GF32>
void launch_lamb_one_by_policy(const cc_plan *p, const StepScalars &s, int32_t *flag, hipStream_t st)
{
    if (p->mem.lamb1 == CC_CACHE_RESIDENT) launch_lamb_one<GF32, Resident>(p, s, flag, st);
    else if (p->mem.lamb1 == CC_CACHE_WRITE_THROUGH) launch_lamb_one<GF32, WriteThrough>(p, s, flag, st);
    else launch_lamb_one<GF32, Streaming>(p, s, flag, st);
}

}  // namespace

int lamb_one_launch(cc_plan *p, const StepScalars &s, int32_t *flag, hipStream_t st)
{
    if (p->grad_f32) launch_lamb_one_by_policy<true>(p, s, flag, st);
    else launch_lamb_one_by_policy<false>(p, s, flag, st);
    return launched("lamb_one_launch_kernel");
}

}  // namespace ccf
