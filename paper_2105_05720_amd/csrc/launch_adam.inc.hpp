// Launches of the fused Adam kernels for one gradient element type (every R, mode, schedule, workgroup size and cache
// policy).  Included by launch_adam_f16.hip and launch_adam_f32.hip, which exist as two sources only so that the two
// element types compile side by side.
#pragma once

#include "plan.hpp"

namespace ccf {

namespace {

// One tensor that does not fit the Infinity Cache, in single-wave pieces (see kFlatPiece).
template <int MODE, bool GF32, class MEM>
void launch_flat_pieces(const DevTensor &t, int R, StepScalars s, FlagScratch *fs, int32_t *flag, hipStream_t st, bool slices_plain = false)
{
    const dim3 grid((unsigned)((t.numel + kFlatPiece - 1) / kFlatPiece)), block(kFlatBlock);
    const unsigned lds = flat_lds(t.numel, R, GF32, std::is_same<MEM, Streaming>::value);
    s.chunk_elems = kFlatPiece;
    if constexpr (std::is_same<MEM, WriteThrough>::value) {
        if (slices_plain) {
            switch (R) {
#define CASE(r) case r: if constexpr (slices_plain_for(r, GF32)) hipLaunchKernelGGL((fused_adam_flat_kernel<r, MODE, kFlatBlock, GF32, 1, MEM, true>), grid, block, lds, st, t, s, fs, flag); break;
                FOR_EACH_R(CASE)
#undef CASE
            }
            return;
        }
    }
    switch (R) {
#define CASE(r) case r: hipLaunchKernelGGL((fused_adam_flat_kernel<r, MODE, kFlatBlock, GF32, 1, MEM>), grid, block, lds, st, t, s, fs, flag); break;
        FOR_EACH_R(CASE)
#undef CASE
    }
}

// A list that stores too much to write through, in the same pieces (see list_in_pieces).
template <int MODE, bool GF32>
void launch_list_pieces(const cc_plan *p, const StepScalars &s, int32_t *flag, hipStream_t st)
{
    const Layout &L = *p->list_pieces;
    const dim3 grid((unsigned)L.chunks * kPiecesPerChunk), block(kFlatBlock);
    const unsigned lds = flat_lds(p->numel, p->R, GF32, true);
    switch (p->R) {
#define CASE(r) case r: if constexpr (pieces_take(r, GF32)) hipLaunchKernelGGL((fused_adam_piece_kernel<r, MODE, GF32, Streaming>), grid, block, lds, st, L.d_tensors, L.d_chunks, s, p->d_flag_scratch, flag); break;
        FOR_EACH_R(CASE)
#undef CASE
    }
}

// One tensor in chunks of kPackedChunk elements whose arguments fit 96 bytes.  False: they do not.
template <int MODE, bool GF32, class MEM>
bool launch_packed(const DevTensor &t, int R, const StepScalars &s, FlagScratch *fs, int32_t *flag, hipStream_t st)
{
    const auto word = [](const void *p) { return (uint64_t)reinterpret_cast<uintptr_t>(p); };
    const uint64_t address[8] = {word(t.w_in), word(t.m_in), word(t.v_in), word(t.w_out), word(t.m_out), word(t.v_out), word(t.w16), word(t.grad[0])};
    uint64_t grad[CC_MAX_R];
    for (int r = 0; r < R; ++r) grad[r] = word(t.grad[r]);
    PackedAdam a;
    if (!pack_adam(address, grad, R, word(flag), word(fs), t.numel, &a)) return false;
    a.inv_div = s.inv_div;
    a.wd = t.wd;
    a.beta1 = (float)s.beta1; a.beta2 = (float)s.beta2;                  // the interface's fp32 values
    a.rc1 = s.rc1; a.rc2 = s.rc2; a.eps = s.eps; a.lr = s.lr;
    const dim3 grid((a.numel + (kPackedChunk - 1)) / kPackedChunk), block(kSmallBlock);
    switch (R) {
#define CASE(r) case r: hipLaunchKernelGGL((fused_adam_packed_kernel<r, MODE, kSmallBlock, GF32, MEM>), grid, block, 0, st, a); break;
        FOR_EACH_R(CASE)
#undef CASE
    }
    return true;
}

template <int MODE, int BLK, bool GF32, class MEM>
void launch_fused_adam_r(const cc_plan *p, const StepScalars &s, int32_t *flag, hipStream_t st)
{
    const Layout &L = p->lay();
    if constexpr (std::is_same<MEM, Streaming>::value)
        if (p->list_pieces) return launch_list_pieces<MODE, GF32>(p, s, flag, st);
    if constexpr (BLK == kBigBlock)
        if (p->flat_adam) return launch_flat_pieces<MODE, GF32, Streaming>(L.host_tensors[(size_t)p->single], p->R, s, p->d_flag_scratch, flag, st);
    if (p->ordered) {
        const dim3 grid(ordered_grid(p)), block(kBigBlock);
        switch (p->R) {
#define CASE(r) case r: hipLaunchKernelGGL((fused_adam_ordered_kernel<r, MODE, kBigBlock, GF32>), grid, block, 0, st, ORDERED_ARGS(p, kSpanAdam), s, p->d_queue, flag); break;
            FOR_EACH_R(CASE)
#undef CASE
        }
        return;
    }
    const dim3 grid((unsigned)L.chunks), block(BLK);
    if (p->single >= 0) {                  // one tensor: no table, descriptor in the kernel arguments
        const DevTensor &t = L.host_tensors[(size_t)p->single];
        if constexpr (!std::is_same<MEM, Resident>::value)
            if (p->flat_pieces && t.numel <= kFlatMaxElems) return launch_flat_pieces<MODE, GF32, MEM>(t, p->R, s, p->d_flag_scratch, flag, st, p->fused.slices_plain);
        if constexpr (BLK == kSmallBlock && !std::is_same<MEM, WriteThrough>::value)
            if (L.chunk_elems == kSmallChunkElems && launch_packed<MODE, GF32, MEM>(t, p->R, s, p->d_flag_scratch, flag, st)) return;
        switch (p->R) {
#define CASE(r) case r: hipLaunchKernelGGL((fused_adam_flat_kernel<r, MODE, BLK, GF32, 2, MEM>), grid, block, 0, st, t, s, p->d_flag_scratch, flag); break;
            FOR_EACH_R(CASE)
#undef CASE
        }
        return;
    }
    const unsigned lds = p->spread_adam ? list_lds(p->numel, p->R, GF32, std::is_same<MEM, Streaming>::value) : 0u;
    if constexpr (std::is_same<MEM, WriteThrough>::value) {
        if (p->fused.slices_plain) {
            switch (p->R) {
#define CASE(r) case r: if constexpr (slices_plain_for(r, GF32)) hipLaunchKernelGGL((fused_adam_kernel<r, MODE, BLK, GF32, 2, MEM, true>), grid, block, lds, st, L.table_tensors(), L.table_chunks(), s, p->d_flag_scratch, flag); break;
                FOR_EACH_R(CASE)
#undef CASE
            }
            return;
        }
    }
    switch (p->R) {
#define CASE(r) case r: hipLaunchKernelGGL((fused_adam_kernel<r, MODE, BLK, GF32, 2, MEM>), grid, block, lds, st, L.table_tensors(), L.table_chunks(), s, p->d_flag_scratch, flag); break;
        FOR_EACH_R(CASE)
#undef CASE
    }
}

template <int BLK, bool GF32, class MEM>
void launch_mode(const cc_plan *p, const StepScalars &s, int32_t *flag, hipStream_t st, int mode)
{
    switch (mode) {
        case 0: launch_fused_adam_r<0, BLK, GF32, MEM>(p, s, flag, st); break;
        case 1: launch_fused_adam_r<1, BLK, GF32, MEM>(p, s, flag, st); break;
        case 2: launch_fused_adam_r<2, BLK, GF32, MEM>(p, s, flag, st); break;
        default: launch_fused_adam_r<3, BLK, GF32, MEM>(p, s, flag, st); break;
    }
}

template <bool GF32>
void launch_fused_adam(const cc_plan *p, const StepScalars &s, int32_t *flag, hipStream_t st, int mode)
{
    BY_BLOCK_MEM(p, p->fused.adam, (launch_mode<BLK, GF32, MEM>(p, s, flag, st, mode)));
}

}  // namespace

}  // namespace ccf
