// Device side of ccfused: streaming kernels for gfx950 (wave64).
//
// Every kernel here is bound by HBM bandwidth: per parameter the fused Adam step moves 2R bytes of fp16
// gradients and 26 bytes of fp32/fp16 state against ~R + 30 scalar flops, so there is no contraction and no
// MFMA.  The shape follows from what the memory system rewards:
//
//   * One workgroup per chunk of one tensor; the chunk table replaces a per-thread search over the scattered
//     tensors (Section 5.4).  The table entry and the tensor descriptor are uniform, so they arrive through
//     scalar loads and every buffer is addressed as scalar base + 32-bit lane offset.
//   * Ownership is chosen so that EVERY access instruction of a wave covers one contiguous span: a lane owns
//     4 consecutive elements per group, i.e. one 16-byte access per fp32 array (1 KiB per wave instruction)
//     and one 8-byte access per fp16 array (512 B per wave instruction).  Letting a lane own 8 consecutive
//     elements instead would split each fp32 row of a wave into two half-filled store instructions, and HBM
//     pays dearly for partially written lines (measured: 2.5 TB/s against 5.8 TB/s for the stores alone).
//   * Two groups per sweep, all loads of both groups issued before the first use, so that each wave keeps
//     2 x (R + 3) independent requests in flight.
//   * The reduced gradient stays in registers (Section 3.3, AllReduce Fuse: the output of the reduction is
//     handed to the computation directly, never through memory).
//   * Large shards run under the ordered persistent schedule (ordered_stream below): one workgroup per compute
//     unit, chunks handed out in table order from one counter, the next chunk's loads in flight while the current
//     one is computed.  What it buys is on the DRAM side: the addresses in flight at any moment form a narrow
//     window that slides through each stream, instead of the wide, drifting set that a grid of independent
//     workgroups produces.  Small shards keep one workgroup per chunk (more parallel start-up, no ticket latency).
#pragma once
// (Kernels that are not templates are `static`: this header is included by several translation units.)

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "ccfused.h"
#include "flag_word.hpp"
#include "meeting.hpp"
#include "occupancy.hpp"
#include "packed_args.hpp"
#include "piece_order.hpp"

namespace ccf {

constexpr uint32_t kStatePack = 4;     // consecutive elements a lane owns per group wherever an fp32 array is written

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// One tensor of the shard as the kernels see it.
struct DevTensor {
    uint64_t numel;
    const float *w_in, *m_in, *v_in;
    float *w_out, *m_out, *v_out;
    uint16_t *w16;
    const void *grad[CC_MAX_R];   // fp16 bit patterns, or fp32 values when the plan says so
    float *gsum;              // unfused pipelines only: fp32 reduced gradient of this tensor
    float wd;
    uint32_t first_chunk;     // position of this tensor's first chunk in the table
    uint32_t num_chunks;
    uint32_t tensor;          // index of this tensor in the plan's list
    uint32_t chunk_index;     // per-chunk copies of the descriptor only (see locate_at): which chunk of the tensor
    uint32_t first_group;     // which group of 64 chunks its first one starts, counted over the shard (see LambMeeting)
};

// Chunk table entry: which tensor, and which chunk_elems-sized piece of it.
struct Chunk {
    uint32_t tensor;
    uint32_t index;
};

// Scalars of one step, precomputed on the host in double and rounded once.
struct StepScalars {
    double inv_div;           // 1 / (loss_scale * (average ? R : 1))
    double beta1, beta2;      // the interface's fp32 values, promoted
    double omb1, omb2;        // 1 - beta, exact in double
    float rc1, rc2;           // 1 / (1 - beta^t)
    float eps, lr;
    uint32_t chunk_elems;
    uint32_t runs;            // one workgroup per chunk: take the chunks in runs per XCD (piece_in_runs)
};

enum : int { kModeGuard = 1, kModeL2 = 2 };

__device__ __forceinline__ bool not_finite(float x) { return !(__builtin_fabsf(x) <= 3.402823466e+38f); }

// Moments of one element from the reduced sum S (Fig. 4a: the m and v updates), each formed in double from the fp32
// inputs and rounded to fp32 once, so that the stored moments are the correctly rounded values of their definitions
// (up to double rounding).  In fp32 the terms would be rounded one by one, and where they cancel (the two terms of
// m', or S / (loss_scale D) against wd w in L2 mode) the result carries those roundings at full size: random cases
// put a few elements at 1.3 x the parity bound that way.  Eight double-precision operations per element, which
// neither the HBM-bound nor the launch-bound kernels notice.
template <int MODE>
__device__ __forceinline__ void moments(float S, float w, float wd, const StepScalars &s, float &m, float &v)
{
    double g = (double)S * s.inv_div;
    if (MODE & kModeL2) g = __builtin_fma((double)wd, (double)w, g);
    m = (float)__builtin_fma(s.beta1, (double)m, s.omb1 * g);
    v = (float)__builtin_fma(s.beta2, (double)v, (s.omb2 * g) * g);
}

// Update direction u from the new moments (Fig. 4a: bias corrections and the quotient), plus decoupled decay.
template <int MODE>
__device__ __forceinline__ float direction(float w, float wd, float m, float v, const StepScalars &s)
{
    const float mh = m * s.rc1;
    const float vh = v * s.rc2;
    // v_sqrt_f32 and v_rcp_f32, each within 1 ulp: the quotient is off by at most ~3 x 2^-24 relative, which moves
    // w by lr |u| 2e-7, two orders below the 2e-6 parity bound; the IEEE sequences cost 20 more instructions per
    // element, which a small (launch-bound) shard pays in full.
    float u = mh * __builtin_amdgcn_rcpf(__builtin_amdgcn_sqrtf(vh) + s.eps);
    if (!(MODE & kModeL2)) u = __builtin_fmaf(wd, w, u);
    return u;
}

// ---- memory access: every buffer is device memory, addressed as uniform base + 32-bit byte offset ----------
#define CCF_GLOBAL __attribute__((address_space(1)))
typedef const CCF_GLOBAL char *gcbytes;
typedef CCF_GLOBAL char *gbytes;

// Base of a chunk inside one of a tensor's arrays (generic pointers from the descriptor become global ones).
__device__ __forceinline__ gcbytes chunk_base(const void *p, uint64_t byte_off) { return (gcbytes)p + byte_off; }
__device__ __forceinline__ gbytes chunk_base(void *p, uint64_t byte_off) { return (gbytes)p + byte_off; }

// Cache policy of a kernel's vector accesses.
//   Streaming:    non-temporal hints on every access.  Right for shards far beyond what the chip holds: the data is
//                 not touched again before it has left every cache (+3 % with one workgroup per chunk, +7 % on the
//                 stores under the ordered schedule).
//   Resident:     plain loads, and stores that are written through to the device's coherence point (the sc1 bit), for
//                 shards whose whole step (inputs and outputs of two consecutive steps, which ping-pong between two
//                 copies) fits the 256 MB Infinity Cache.  The next step then finds what this one wrote on chip, and
//                 no dirty lines are left in the L2s for the end of the kernel to write back.  On the memory pattern
//                 of a 2^20-element step: 5.2 us, against 6.6-6.8 us for every combination of plain or non-temporal
//                 loads with plain or non-temporal stores on the same machine.
//   WriteThrough: non-temporal loads with the written-through stores, for shards of a few times the Infinity Cache.
//                 Memory pattern of a 2^24-element step with four slices (570 MB): 72 us, against 93 us for Streaming
//                 and 102 us for Resident; at 2^20 elements it is the slowest of the three (7.1 us), at 2^26 it is 2 %
//                 behind Streaming.
// The compiler has no spelling for a vector store with the sc1 bit, hence the asm; the s_nop behind each store is the
// wait the hardware asks for between a store of more than 64 bits and a vector instruction that overwrites the
// registers holding its data, which the compiler inserts for its own stores but cannot for one it does not see.
struct Streaming { static constexpr bool kLoadNonTemporal = true, kStoreThrough = false; };
struct Resident { static constexpr bool kLoadNonTemporal = false, kStoreThrough = true; };
struct WriteThrough { static constexpr bool kLoadNonTemporal = true, kStoreThrough = true; };
// LAMB's first sweep only: WriteThrough, but the weights, which the second sweep reads again, by plain loads (see fused_policies).
struct WeightsKept : WriteThrough {};
template <class Mem> struct ReadAgain { typedef Mem Policy; };
template <> struct ReadAgain<WeightsKept> { typedef Resident Policy; };

template <class Mem> __device__ __forceinline__ f32x4 ld_f32x4(gcbytes b, uint32_t off)
{
    if (Mem::kLoadNonTemporal) return __builtin_nontemporal_load((const CCF_GLOBAL f32x4 *)(b + off));
    return *(const CCF_GLOBAL f32x4 *)(b + off);
}
template <class Mem> __device__ __forceinline__ f16x4 ld_f16x4(gcbytes b, uint32_t off)
{
    if (Mem::kLoadNonTemporal) return __builtin_nontemporal_load((const CCF_GLOBAL f16x4 *)(b + off));
    return *(const CCF_GLOBAL f16x4 *)(b + off);
}
template <class Mem> __device__ __forceinline__ void st_f32x4(gbytes b, uint32_t off, f32x4 x)
{
    if (!Mem::kStoreThrough) __builtin_nontemporal_store(x, (CCF_GLOBAL f32x4 *)(b + off));
    else asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" : : "v"(b + off), "v"(x) : "memory");
}
template <class Mem> __device__ __forceinline__ void st_f16x4(gbytes b, uint32_t off, f16x4 x)
{
    if (!Mem::kStoreThrough) __builtin_nontemporal_store(x, (CCF_GLOBAL f16x4 *)(b + off));
    else asm volatile("global_store_dwordx2 %0, %1, off sc1\n\ts_nop 1" : : "v"(b + off), "v"(x) : "memory");
}
__device__ __forceinline__ float ld_f32(gcbytes b, uint32_t off) { return *(const CCF_GLOBAL float *)(b + off); }
__device__ __forceinline__ float ld_f16(gcbytes b, uint32_t off) { return (float)*(const CCF_GLOBAL _Float16 *)(b + off); }
__device__ __forceinline__ void st_f32(gbytes b, uint32_t off, float x) { *(CCF_GLOBAL float *)(b + off) = x; }

// fp32 -> fp16, round to nearest even, of the fp32 value as stored.  The empty asm pins x in a register so
// that the compiler cannot merge the conversion with the fma that produced x into one mixed-precision fma
// (v_fma_mixlo_f16 rounds the exact product-sum straight to fp16, which can differ from rounding the fp32
// result by one fp16 ulp).
__device__ __forceinline__ _Float16 to_half(float x)
{
    asm volatile("" : "+v"(x));
    return (_Float16)x;
}
__device__ __forceinline__ void st_f16(gbytes b, uint32_t off, float x) { *(CCF_GLOBAL _Float16 *)(b + off) = to_half(x); }

template <class Mem> __device__ __forceinline__ void ld_f32x4(gcbytes b, uint32_t off, float (&x)[4])
{
    const f32x4 t = ld_f32x4<Mem>(b, off);
    x[0] = t.x; x[1] = t.y; x[2] = t.z; x[3] = t.w;
}
template <class Mem> __device__ __forceinline__ void st_f32x4(gbytes b, uint32_t off, const float (&x)[4])
{
    st_f32x4<Mem>(b, off, f32x4{x[0], x[1], x[2], x[3]});
}
template <class Mem> __device__ __forceinline__ void st_f16x4(gbytes b, uint32_t off, const float (&x)[4])
{
    st_f16x4<Mem>(b, off, f16x4{to_half(x[0]), to_half(x[1]), to_half(x[2]), to_half(x[3])});
}

// ---- where a workgroup works -----------------------------------------------------------------------------------
// Descriptors and table entries are constant while a kernel runs, and are read through pointers that say so: behind the
// flag's atomic and the stores written in assembly the compiler otherwise takes them for memory that may change, and may
// fetch them with vector loads and keep every buffer's address in vector registers.  Vector registers of the list's fused
// Adam kernel with addresses there / in scalar registers (-Rpass-analysis=kernel-resource-usage): R = 8 written through
// 118 / 104, non-temporal 118 / 114; R = 16 219 / 140 and 219 / 149.
#define CCF_CONSTANT __attribute__((address_space(4)))
typedef const CCF_CONSTANT DevTensor *Descriptor;
typedef const CCF_CONSTANT struct Chunk *ChunkEntry;

struct Where {
    Descriptor t;
    uint32_t tensor;          // index of t in the plan's tensor list
    uint32_t slot;            // position of the chunk in tensor order (first_chunk + index): where its LAMB partials go
    uint32_t index;           // which chunk of the tensor
    uint64_t base;            // first element of the chunk inside the tensor
    uint32_t len;             // elements in this chunk (the tensor's last chunk may be short)
};

constexpr int kLineOfGrads = 7;
// Fields from all over the descriptor before the first is looked at, so that its cache lines arrive together.  Left
// alone the compiler asks for the length, waits, and then asks for the rest.  Descriptors are 224 bytes apart, so every
// other one starts in the middle of a 64-byte line; the length, grad[0], grad[7] and the index lie in all of the lines
// that up to eight slices need.  With more, an entry that starts on a line gets the line of grad[8] to grad[15] later.
__device__ __forceinline__ uint32_t all_lines(Where &wh)
{
    uint32_t own_index = wh.t->chunk_index, own_tensor = wh.t->tensor;
    asm volatile("" : "+s"(own_index), "+s"(own_tensor) : "s"(wh.t->numel), "s"(wh.t->grad[0]), "s"(wh.t->grad[kLineOfGrads]));
    wh.tensor = own_tensor;
    return own_index;
}

// What is left to derive once the descriptor and the chunk's index are known.
__device__ __forceinline__ void finish_where(Where &wh, uint32_t chunk_elems)
{
    wh.slot = wh.t->first_chunk + wh.index;
    wh.base = (uint64_t)wh.index * chunk_elems;
    const uint64_t rem = wh.t->numel - wh.base;
    wh.len = rem < chunk_elems ? (uint32_t)rem : chunk_elems;
}

// Table entry `entry` (uniform over the workgroup) resolved through the tensor descriptor.
__device__ __forceinline__ Where locate_at(const DevTensor *__restrict__ tensors, const Chunk *__restrict__ chunks,
                                           uint32_t entry, uint32_t chunk_elems)
{
    const ChunkEntry c = (ChunkEntry)chunks + entry;
    Where wh;
    wh.tensor = c->tensor;
    wh.index = c->index;
    wh.t = (Descriptor)tensors + wh.tensor;
    finish_where(wh, chunk_elems);
    return wh;
}

// The chunk of this workgroup under the one-workgroup-per-chunk launches.  Plans of few chunks pass chunks == nullptr
// and, as `tensors`, one copy of the descriptor per chunk with the chunk's index in it: the workgroup then knows where
// its data is after one trip to memory instead of two dependent ones (entry, then descriptor): 2-4 % of a launch-bound
// step (same machine, with / without: 4.70 / 4.90 us on 398 tensors in 571 chunks, 9.60 / 9.90 us on 10 tensors in
// 1280 chunks).
constexpr uint32_t kChunkRunLog2 = 5;
// LAST_FIRST: a second sweep over a shard bound by HBM takes the chunks from the other end, and so finds on chip what the
// first sweep touched last.  LAMB, R = 8, from the same end / from the other: 353 / 350.5 us at 42 M elements of the BERT-Large
// list, 482 / 475.5 at 56 M, R = 1 one tensor of 40 M elements 249.5 / 245.5; up to 21 M elements within 1 %.  The ordered
// schedule gained nothing from it (336 M elements: 2808 / 2865 us, runs 2 % apart) and keeps the table's order.
template <bool LAST_FIRST = false>
__device__ __forceinline__ Where locate(const DevTensor *__restrict__ tensors, const Chunk *__restrict__ chunks, const StepScalars &s)
{
    uint32_t entry = (uint32_t)__builtin_amdgcn_readfirstlane((int)(s.runs ? piece_in_runs<kChunkRunLog2>(blockIdx.x, gridDim.x) : blockIdx.x));
    if (LAST_FIRST && s.runs) entry = gridDim.x - 1 - entry;
    uint32_t tensor = entry, index = 0;
    if (chunks != nullptr) {
        const ChunkEntry c = (ChunkEntry)chunks + entry;
        tensor = c->tensor;
        index = c->index;
    }
    Where wh;
    wh.t = (Descriptor)tensors + tensor;
    const uint32_t own_index = all_lines(wh);
    wh.index = chunks != nullptr ? index : own_index;
    finish_where(wh, s.chunk_elems);
    return wh;
}

// The overflow flag is produced by the same launch that does the work, with no clearing launch in front of it and
// with nothing on the path between a wave's loads and its stores.
//
// What has to happen: the caller's flag must read 0 after a launch in which no wave saw an inf/NaN and 1 otherwise,
// and the scratch words must be ready for the next launch.  Counting FINISHED workgroups (the obvious way to find
// "the last one", who then writes the flag) puts two dependent atomic round trips behind the last wave's loads, and a
// returning atomic issued after the stores is only seen once those stores are acknowledged (the memory counter is
// in order): measured 0.9-1.7 us on a 6 us step.  So ARRIVALS are counted instead:
//
//   * Lane 0 of every wave adds 1 to one of kFlagSlots slot words as its very first act, before any load.  The
//     result comes back while the loads are in flight.  The high half of a slot word is the launch's phase p (the
//     same in every slot between launches), so the one atomic tells a wave p and whether it is the last arrival in
//     its slot.  That wave puts the slot back to (p+1, 0) and adds 1 to the top word; the wave that completes the top
//     word is the last arrival of the launch: every wave has arrived, none will touch the counters again, so it can
//     zero the top word and move the slots this launch did not use to p+1 as well.
//   * The last arrival clears the caller's flag with a returning exchange issued before its own update and stores,
//     and, behind its stores, once that exchange has returned (so the 0 has been performed at the device's coherence
//     point), exchanges the state word to (p+1, CLEARED).  If this second exchange returns (p+1, BAD), a wave had
//     reported an inf/NaN before, and the last arrival sets the flag to 1 itself.  (A release on the second exchange
//     would state the same order in the language's terms, but costs a write-back of the whole L2 in the middle of
//     the kernel on the one wave that everybody ends up waiting for: measured +0.7 to +1.3 us per step.  The order is
//     enforced in the source instead: the second exchange takes an operand that depends on the first one's result.)
//   * A wave that saw an inf/NaN (rare) moves the state word to (p+1, BAD) with a compare-exchange loop, unless it
//     finds (p+1, CLEARED) there: then the flag's 0 was performed before, and it stores 1 into the flag itself.
//     Either the last arrival's exchange comes first in the state word's modification order, and the reporting wave
//     sees CLEARED and writes 1 after the 0; or the report comes first, and the exchange returns it.  Both can write 1.
//   * Values of older launches in the state word carry another phase and are ignored, so nothing has to be reset at
//     the end of a launch, which is what would need a count of finished waves.
//
// Nothing waits on another wave.  Per launch every wave issues one atomic; one wave per slot issues three more; one
// wave issues the handful around the flag.  Phases are 32 bits and wrap; a report that is exactly 2^32 launches old
// would be taken for a new one.
constexpr uint32_t kFlagSlots = 128;
struct FlagScratch {
    struct alignas(128) Line { unsigned long long word; } slot[kFlagSlots], top, state;
};
struct FlagWords {
    unsigned long long *state;
    int32_t *flag;
    __device__ __forceinline__ unsigned long long read() const { return __hip_atomic_load(state, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT); }
    __device__ __forceinline__ unsigned long long exchange(unsigned long long x) const { return __hip_atomic_exchange(state, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
    __device__ __forceinline__ bool replace(unsigned long long &cur, unsigned long long x) const
    {
        return __hip_atomic_compare_exchange_strong(state, &cur, x, __ATOMIC_ACQ_REL, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ __forceinline__ void raise() const { __hip_atomic_store(flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
};

template <int BLOCK>
struct FlagCount {
    unsigned long long prev = 0ull, tprev = 0ull;
    uint32_t slot = 0, in_slot = 0, used = 0;
    int32_t flag_before = 0;
    bool slot_last = false, launch_last = false;

    __device__ __forceinline__ bool counting_lane() const { return (threadIdx.x & 63u) == 0u; }
    __device__ __forceinline__ uint32_t tag() const { return (uint32_t)(prev >> 32) + 1u; }          // this launch's p + 1

    // First act of a kernel: the wave's arrival.  Nothing is waited for here.
    __device__ __forceinline__ void arrive(FlagScratch *fs) { arrive(fs, gridDim.x); }
    __device__ __forceinline__ void arrive(FlagScratch *fs, uint32_t workgroups)
    {
        if (counting_lane()) {
            constexpr uint32_t kWaves = BLOCK / 64;
            const uint32_t waves = workgroups * kWaves;
            const uint32_t me = blockIdx.x * kWaves + (threadIdx.x >> 6);
            slot = me % kFlagSlots;
            in_slot = (waves - slot + kFlagSlots - 1) / kFlagSlots;      // waves w with w % kFlagSlots == slot
            used = waves < kFlagSlots ? waves : kFlagSlots;
            prev = atomicAdd(&fs->slot[slot].word, 1ull);
        }
    }
    // Once the arrival's result is needed (behind the issue of the loads): the last arrival in a slot moves on to the top word.
    __device__ __forceinline__ void slot_level(FlagScratch *fs)
    {
        if (counting_lane()) {
            slot_last = (uint32_t)prev == in_slot - 1;
            if (slot_last) {
                atomicExch(&fs->slot[slot].word, (unsigned long long)tag() << 32);
                tprev = atomicAdd(&fs->top.word, 1ull);
            }
        }
    }
    // Before the wave's stores: the last arrival of the launch tidies the counters and starts clearing the flag.  Every
    // lane of the wave calls this.  The slots a small launch did not use are moved on by all 64 lanes at once, behind
    // the flag's exchange: one lane doing it slot by slot, in front of the exchange, cost a launch of one workgroup 2 us.
    __device__ __forceinline__ void top_level(FlagScratch *fs, int32_t *flag)
    {
        if (counting_lane() && slot_last) {
            launch_last = (uint32_t)tprev == used - 1;
            if (launch_last) {
                atomicExch(&fs->top.word, 0ull);
                flag_before = __hip_atomic_exchange(flag, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        if (__builtin_amdgcn_ballot_w64(launch_last) != 0ull) {            // uniform: this wave holds the last arrival
            const uint32_t first_unused = (uint32_t)__builtin_amdgcn_readfirstlane((int)used);
            const uint32_t next_tag = (uint32_t)__builtin_amdgcn_readfirstlane((int)tag());
            for (uint32_t k = first_unused + (threadIdx.x & 63u); k < kFlagSlots; k += 64u)
                atomicExch(&fs->slot[k].word, (unsigned long long)next_tag << 32);
        }
    }
    // After the wave's stores have been issued: reports.
    __device__ __forceinline__ void finish(bool bad, FlagScratch *fs, int32_t *flag)
    {
        const bool any = __builtin_amdgcn_ballot_w64(bad) != 0ull;
        if (counting_lane()) {
            if (launch_last) {
                uint32_t mine = tag();
                asm volatile("" : "+v"(mine) : "v"(flag_before));     // not before the flag's exchange has returned
                flag_cleared(FlagWords{&fs->state.word, flag}, mine);
            }
            if (any) report(fs, flag);
        }
    }
    // What a wave finds later than that, by its counting lane.
    __device__ __forceinline__ void report(FlagScratch *fs, int32_t *flag) const { flag_report(FlagWords{&fs->state.word, flag}, tag()); }
    // Everything behind the arrival at once, for kernels that do not place the stages themselves.
    __device__ __forceinline__ void settle(bool bad, FlagScratch *fs, int32_t *flag)
    {
        slot_level(fs);
        top_level(fs, flag);
        finish(bad, fs, flag);
    }
};

// Only for a plan without any chunk: nothing else would write the flag.
[[maybe_unused]] static __global__ void clear_flag_kernel(int32_t *flag) { *flag = 0; }

// ---- the streaming skeleton --------------------------------------------------------------------------------------
// An Op describes one kernel's per-element work:
//   static constexpr uint32_t kPack;               consecutive elements a lane owns per group
//   struct Regs;                                   registers of one group (kPack elements of this lane)
//   void load(Regs&, uint32_t e) const;            vector loads of elements e .. e+kPack-1 of the chunk
//   void compute(Regs&);                           arithmetic on the group
//   void store(const Regs&, uint32_t e) const;     vector stores
//   void single(uint32_t j);                       one element, scalar accesses (ragged end of a tensor)
// and, where its chunks go through a Sweep, compute() in two parts:
//   void reduce(Regs&);                            what the overflow flag needs (sweep_and_publish only)
//   void update(Regs&);                            the rest; called for lanes whose pack is inside the chunk only
// A sweep is GROUPS groups, BLOCK*kPack elements apart: it issues the loads of all of them, then computes and stores.

// The last len % kPack elements of a chunk: one lane each, so that they cost one trip to memory together (one lane going
// through three of them cost three).
template <class Op>
__device__ __forceinline__ void ragged_end(Op &op, uint32_t len)
{
    constexpr uint32_t kMask = Op::kPack - 1;
    if (threadIdx.x < (len & kMask)) op.single((len & ~kMask) + threadIdx.x);
}

// A chunk of any length: full sweeps, then group by group.
template <int BLOCK, class Op, int GROUPS = 2>
__device__ __forceinline__ void stream_chunk(Op &op, uint32_t len)
{
    constexpr uint32_t kLanePack = Op::kPack;      // consecutive elements a lane owns per group
    constexpr uint32_t kGroup = BLOCK * kLanePack;
    constexpr uint32_t kSweep = GROUPS * kGroup;
    const uint32_t lane_e = threadIdx.x * kLanePack;
    uint32_t s0 = 0;
    for (; s0 + kSweep <= len; s0 += kSweep) {
        typename Op::Regs x[GROUPS];
#pragma unroll
        for (int g = 0; g < GROUPS; ++g) op.load(x[g], s0 + g * kGroup + lane_e);
        __builtin_amdgcn_sched_barrier(0);         // keep all loads of the sweep ahead of the first use
#pragma unroll
        for (int g = 0; g < GROUPS; ++g) {
            op.compute(x[g]);
            op.store(x[g], s0 + g * kGroup + lane_e);
        }
    }
    for (uint32_t e = s0 + lane_e; e + kLanePack <= len; e += kGroup) {
        typename Op::Regs a;
        op.load(a, e);
        op.compute(a);
        op.store(a, e);
    }
    ragged_end(op, len);
}

// A chunk of at most one sweep (the launch shapes the plans use), in the same steps whether it is full or not: a lane
// past the end loads the chunk's last whole pack once more, so that all loads are issued together and without branches,
// and stores nothing.  (Every tensor ends in a short chunk and most tensors of a list are one; group by group they cost a
// trip to memory per group, with the flag's three behind them.)  Needs at least one whole pack.
template <int BLOCK, int GROUPS, class Op>
struct Sweep {
    static constexpr uint32_t kGroup = BLOCK * Op::kPack;
    typename Op::Regs x[GROUPS];
    __device__ __forceinline__ static uint32_t first(int g) { return g * kGroup + threadIdx.x * Op::kPack; }
    __device__ __forceinline__ static bool mine(int g, uint32_t len) { return first(g) + Op::kPack <= len; }
    __device__ __forceinline__ void load(const Op &op, uint32_t len)
    {
        const uint32_t last = (len & ~(Op::kPack - 1u)) - Op::kPack;
#pragma unroll
        for (int g = 0; g < GROUPS; ++g) op.load(x[g], first(g) < last ? first(g) : last);
    }
    __device__ __forceinline__ void update_and_store(Op &op, uint32_t len)
    {
#pragma unroll
        for (int g = 0; g < GROUPS; ++g)
            if (mine(g, len)) { op.update(x[g]); op.store(x[g], first(g)); }
        ragged_end(op, len);
    }
};

// One workgroup per chunk, for an Op that raises the flag.  `fc` has arrived already (first act of the kernel).  The
// stages of the count are placed where their results are free: the slot level behind the issue of the loads, the top
// level behind the sums, the reports behind the stores.  The waves of a workgroup never wait for each other here.
template <int BLOCK, int GROUPS, class Op>
__device__ __forceinline__ void sweep_and_publish(Op &op, uint32_t len, FlagCount<BLOCK> &fc, FlagScratch *fs, int32_t *flag)
{
    typedef Sweep<BLOCK, GROUPS, Op> S;
    if (len >= Op::kPack && len <= GROUPS * S::kGroup) {
        S sw;
        sw.load(op, len);
        __builtin_amdgcn_sched_barrier(0);
        fc.slot_level(fs);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int g = 0; g < GROUPS; ++g) op.reduce(sw.x[g]);
        fc.top_level(fs, flag);
        __builtin_amdgcn_sched_barrier(0);
        sw.update_and_store(op, len);
        __builtin_amdgcn_sched_barrier(0);
        fc.finish(op.bad, fs, flag);
    } else {
        stream_chunk<BLOCK, Op, GROUPS>(op, len);
        fc.settle(op.bad, fs, flag);
    }
}

// One workgroup per chunk, for an Op whose loads need nothing that the rest of the kernel waits for: they are issued
// first, then ready() finds out what the arithmetic needs, or returns false to leave without a store.
template <int BLOCK, int GROUPS, class Op, class Ready>
__device__ __forceinline__ void sweep_when_ready(Op &op, uint32_t len, Ready ready)
{
    typedef Sweep<BLOCK, GROUPS, Op> S;
    if (len >= Op::kPack && len <= GROUPS * S::kGroup) {
        S sw;
        sw.load(op, len);
        __builtin_amdgcn_sched_barrier(0);
        if (!ready()) return;
        sw.update_and_store(op, len);
    } else {
        if (!ready()) return;
        stream_chunk<BLOCK, Op, GROUPS>(op, len);
    }
}

// ---- the ordered persistent schedule -------------------------------------------------------------------------------
// gridDim.x workgroups (one per compute unit) share the chunk table through one counter.  The table is cut into
// blocks of `span` consecutive entries.  Workgroup b starts with blocks b and b + G (G = gridDim.x) and then takes
// block 2G + ticket, ticket = atomic increment of `next`: blocks are started in table order by whichever workgroup
// is free, so the chunks in flight are always ~2G span consecutive ones.  (A counter that every workgroup of the
// device increments serves about one ticket per 12 ns; span is chosen per kernel so that a ticket covers enough
// bytes for that not to matter.)  The table lists every full chunk first (nfull of them, in address order) and
// the short last chunks of tensors behind them; full chunks go through a two-stage pipeline (loads of the next
// chunk are issued before the current chunk is computed and stored), the few short ones through stream_chunk.
// Nothing waits on another workgroup: a workgroup leaves when its entries are past the table, so the grid drains
// whatever its size.  `done` counts finished workgroups in its low half and those that saw an inf/NaN in its high
// half (one atomic, so no fence has to order two words); the workgroup that completes the count writes the
// caller's flag and zeroes the queue for the next launch.
struct WorkQueue {
    struct alignas(128) Next { uint32_t v; } next;
    struct alignas(128) Done { unsigned long long v; } done;
};

// The increasing sequence of table entries one workgroup works through.  The ticket for the block after the next
// one is requested when a block is entered and only looked at when that later block is entered, a block's worth of
// work later; the one wave that issues the atomic waits for it there and then, the others never do.  Its value
// reaches them through LDS (two slots used in turn: one barrier per block).
struct Entries {
    WorkQueue *q;
    uint32_t *slots;          // LDS, 2 words
    uint32_t span, blk, j, second, ticket;
    bool second_pending;      // the workgroup's second block (blockIdx.x + gridDim.x) has not been entered yet
    int turn;
    __device__ __forceinline__ void init(WorkQueue *queue, uint32_t *lds_slots, uint32_t span_)
    {
        q = queue; slots = lds_slots; span = span_;
        blk = blockIdx.x; second = blockIdx.x + gridDim.x;    // the two blocks every workgroup owns without asking
        second_pending = true;
        j = 0; turn = 0; ticket = 0;
    }
    // every thread of the workgroup calls next() at the same point
    __device__ __forceinline__ uint32_t next()
    {
        if (j == span) {                                      // enter the next block
            j = 0;
            if (second_pending) {
                blk = second;
                second_pending = false;
            } else {
                if (threadIdx.x == 0) slots[turn] = 2 * gridDim.x + ticket;
                __syncthreads();
                blk = (uint32_t)__builtin_amdgcn_readfirstlane((int)slots[turn]);
                turn ^= 1;
            }
            if (threadIdx.x == 0) ticket = atomicAdd(&q->next.v, 1u);      // for the block after the next one
        }
        return blk * span + j++;
    }
};

// An Op used here also provides   template <int BLOCK> void end_chunk(uint32_t slot);   called once per chunk after
// its last store (LAMB phase 1 writes the chunk's partial sums there; the others do nothing).
// bind(op, entry) points op at table entry `entry` and returns its Where.
template <int BLOCK, int GROUPS, class Op, class Bind>
__device__ __forceinline__ void ordered_stream(Op &opa, Op &opb, Bind bind, uint32_t nfull, uint32_t nchunks, uint32_t span,
                                               WorkQueue *q)
{
    __shared__ uint32_t ticket_slots[2];
    constexpr uint32_t kGroup = BLOCK * Op::kPack;
    const uint32_t lane_e = threadIdx.x * Op::kPack;
    Entries en;
    en.init(q, ticket_slots, span);
    uint32_t e = en.next(), n = en.next();         // current and next entry, e < n
    if (e < nfull) {
        typename Op::Regs xa[GROUPS], xb[GROUPS];
        Where wa = bind(opa, e), wb;
#pragma unroll
        for (int g = 0; g < GROUPS; ++g) opa.load(xa[g], g * kGroup + lane_e);
        while (true) {
            if (n < nfull) {                       // past the full chunks there is nothing to fetch ahead
                wb = bind(opb, n);
#pragma unroll
                for (int g = 0; g < GROUPS; ++g) opb.load(xb[g], g * kGroup + lane_e);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int g = 0; g < GROUPS; ++g) { opa.compute(xa[g]); opa.store(xa[g], g * kGroup + lane_e); }
            opa.template end_chunk<BLOCK>(wa.slot);
            __builtin_amdgcn_sched_barrier(0);
            const uint32_t n2 = en.next();
            if (n >= nfull) { e = n; n = n2; break; }
            if (n2 < nfull) {
                wa = bind(opa, n2);
#pragma unroll
                for (int g = 0; g < GROUPS; ++g) opa.load(xa[g], g * kGroup + lane_e);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int g = 0; g < GROUPS; ++g) { opb.compute(xb[g]); opb.store(xb[g], g * kGroup + lane_e); }
            opb.template end_chunk<BLOCK>(wb.slot);
            __builtin_amdgcn_sched_barrier(0);
            e = n2;
            n = en.next();
            if (e >= nfull) break;
        }
    }
    while (e < nchunks) {                          // short chunks, one at a time
        const Where wh = bind(opa, e);
        stream_chunk<BLOCK, Op, GROUPS>(opa, wh.len);
        opa.template end_chunk<BLOCK>(wh.slot);
        e = n;
        n = en.next();
    }
}

// Last act of a workgroup under the ordered schedule: count itself (and whether it saw an inf/NaN); the workgroup
// that completes the count writes the flag (RAISE) and zeroes the queue.
// Why `next` is exactly 0 when the next launch starts: every increment of `next` is issued by thread 0 of some
// workgroup (Entries::next), the same thread that later adds to `done` here, so the increment is sequenced before
// that add.  The add releases and acquires at device scope: the add of the workgroup that completes the count reads
// from the release sequence formed by all the earlier adds, hence every increment of `next` by any workgroup happens
// before the exchange below, which is therefore the last modification of `next` in this launch, also for a
// workgroup whose last ticket was requested but never looked at.  One such add per workgroup per launch costs nothing.
template <bool RAISE>
__device__ __forceinline__ void leave_queue(bool bad, WorkQueue *q, int32_t *flag)
{
    const int any = RAISE ? __syncthreads_or(bad ? 1 : 0) : 0;
    if (threadIdx.x == 0) {
        const unsigned long long mine = 1ull | (any ? (1ull << 32) : 0ull);
        const unsigned long long prev = __hip_atomic_fetch_add(&q->done.v, mine, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
        if ((uint32_t)prev == gridDim.x - 1) {
            if (RAISE) *flag = ((prev + mine) >> 32) != 0ull ? 1 : 0;
            atomicExch(&q->done.v, 0ull);
            atomicExch(&q->next.v, 0u);
        }
    }
}

// The gradient source of a kernel: R slices reduced in registers in fixed rank order; the reduced value is an fp32.
// The slices are fp16 (fp16 -> fp32 is exact, subnormals included; 8 bytes per lane and slice) or fp32 (16 bytes per
// lane and slice); either way the terms are added in double and rounded to fp32 once (see below).
// The unfused pipelines read the fp32 sum that a reduce kernel stored instead (GradSum).
template <int R, bool F32, class MemT = Streaming>
struct GradSlices;

template <int R, class MemT>
struct GradSlices<R, false, MemT> {
    typedef MemT Mem;
    gcbytes g[R];
    struct Regs { f16x4 g[R]; };
    template <class T> __device__ __forceinline__ void init(T t, uint64_t base)
    {
#pragma unroll
        for (int r = 0; r < R; ++r) g[r] = chunk_base(t->grad[r], base * 2);
    }
    __device__ __forceinline__ void load(Regs &x, uint32_t e) const
    {
#pragma unroll
        for (int r = 0; r < R; ++r) x.g[r] = ld_f16x4<Mem>(g[r], e * 2);
    }
    // The sum is formed in double and rounded to fp32 once, in rank order.  Up to 16 fp16 values add exactly in double,
    // so S is the correctly rounded sum whatever the order.  An fp32 running sum is exact only while every partial sum
    // stays below 1 (fp16 values are multiples of 2^-24); with loss-scaled gradients of magnitude ~1 a small addend
    // loses its low bits against a large partial sum (up to 2^-22 absolute per add), and where the slices cancel to
    // |S| ~ 1e-3 that is a relative error of 1e-4 in the reduced gradient.  On the few elements per 10^8 where the
    // unscaled gradient is also comparable with epsilon, u = g/(|g| + eps) turns it into an error of w of 1.8 x the
    // 2e-6 parity bound (measured on the 80 M element embedding of the GPT-2 list).
    __device__ __forceinline__ void sum(const Regs &x, float (&S)[4]) const
    {
        double a = (double)(float)x.g[0].x, b = (double)(float)x.g[0].y, c = (double)(float)x.g[0].z, d = (double)(float)x.g[0].w;
#pragma unroll
        for (int r = 1; r < R; ++r) {
            a += (double)(float)x.g[r].x; b += (double)(float)x.g[r].y; c += (double)(float)x.g[r].z; d += (double)(float)x.g[r].w;
        }
        S[0] = (float)a; S[1] = (float)b; S[2] = (float)c; S[3] = (float)d;
    }
    // One element: loads, and their sum.
    struct One { _Float16 g[R]; };
    __device__ __forceinline__ void load1(One &x, uint32_t j) const
    {
#pragma unroll
        for (int r = 0; r < R; ++r) x.g[r] = *(const CCF_GLOBAL _Float16 *)(g[r] + j * 2);
    }
    __device__ __forceinline__ static float sum1(const One &x)
    {
        double S = (double)(float)x.g[0];
#pragma unroll
        for (int r = 1; r < R; ++r) S += (double)(float)x.g[r];
        return (float)S;
    }
    __device__ __forceinline__ float sum1(uint32_t j) const
    {
        One x;
        load1(x, j);
        return sum1(x);
    }
};

template <int R, class MemT>
struct GradSlices<R, true, MemT> {
    typedef MemT Mem;
    gcbytes g[R];
    struct Regs { f32x4 g[R]; };
    template <class T> __device__ __forceinline__ void init(T t, uint64_t base)
    {
#pragma unroll
        for (int r = 0; r < R; ++r) g[r] = chunk_base(t->grad[r], base * 4);
    }
    __device__ __forceinline__ void load(Regs &x, uint32_t e) const
    {
#pragma unroll
        for (int r = 0; r < R; ++r) x.g[r] = ld_f32x4<Mem>(g[r], e * 4);
    }
    // fp32 slices are added in double and rounded to fp32 once: an fp32 running sum would carry up to
    // (R-1) 2^-24 max|g| of rounding, which a near-zero sum turns into a large relative error of g^2 and, through
    // elements with a small second moment, into an error of w above the 2e-6 bar.  16 fp64 operations per
    // element stay far below the memory time.  A finite sum that does not fit fp32 becomes inf and raises the flag.
    __device__ __forceinline__ void sum(const Regs &x, float (&S)[4]) const
    {
        double a = x.g[0].x, b = x.g[0].y, c = x.g[0].z, d = x.g[0].w;
#pragma unroll
        for (int r = 1; r < R; ++r) { a += (double)x.g[r].x; b += (double)x.g[r].y; c += (double)x.g[r].z; d += (double)x.g[r].w; }
        S[0] = (float)a; S[1] = (float)b; S[2] = (float)c; S[3] = (float)d;
    }
    struct One { float g[R]; };
    __device__ __forceinline__ void load1(One &x, uint32_t j) const
    {
#pragma unroll
        for (int r = 0; r < R; ++r) x.g[r] = ld_f32(g[r], j * 4);
    }
    __device__ __forceinline__ static float sum1(const One &x)
    {
        double S = x.g[0];
#pragma unroll
        for (int r = 1; r < R; ++r) S += (double)x.g[r];
        return (float)S;
    }
    __device__ __forceinline__ float sum1(uint32_t j) const
    {
        One x;
        load1(x, j);
        return sum1(x);
    }
};

template <class MemT = Streaming>
struct GradSum {
    typedef MemT Mem;
    gcbytes s;
    struct Regs { float s[4]; };
    template <class T> __device__ __forceinline__ void init(T t, uint64_t base) { s = chunk_base((const void *)t->gsum, base * 4); }
    __device__ __forceinline__ void load(Regs &x, uint32_t e) const { ld_f32x4<Mem>(s, e * 4, x.s); }
    __device__ __forceinline__ void sum(const Regs &x, float (&S)[4]) const { S[0] = x.s[0]; S[1] = x.s[1]; S[2] = x.s[2]; S[3] = x.s[3]; }
    __device__ __forceinline__ float sum1(uint32_t j) const { return ld_f32(s, j * 4); }
};

// The reduced sum as an fp16 all-reduce hands it over: fp16 values in the first half of the tensor's sum buffer.
template <class MemT = Streaming>
struct GradSumHalf {
    typedef MemT Mem;
    gcbytes s;
    struct Regs { f16x4 s; };
    template <class T> __device__ __forceinline__ void init(T t, uint64_t base) { s = chunk_base((const void *)t->gsum, base * 2); }
    __device__ __forceinline__ void load(Regs &x, uint32_t e) const { x.s = ld_f16x4<Mem>(s, e * 2); }
    __device__ __forceinline__ void sum(const Regs &x, float (&S)[4]) const { S[0] = (float)x.s.x; S[1] = (float)x.s.y; S[2] = (float)x.s.z; S[3] = (float)x.s.w; }
    __device__ __forceinline__ float sum1(uint32_t j) const { return ld_f16(s, j * 2); }
};

// ---------------------------------------------------------------------------------------------------
// Adam: reduce (or read the reduced sum) + moments + weight update (+ fp16 emission when fused).
// One pass, 2R + 26 bytes per parameter when fused.
// ---------------------------------------------------------------------------------------------------
template <class Grad, int MODE, bool EMIT16, class Mem = typename Grad::Mem>
struct AdamOp {
    static constexpr uint32_t kPack = kStatePack;
    Grad grad;
    gcbytes w_in, m_in, v_in;
    gbytes w_out, m_out, v_out, w16;
    StepScalars s;
    float wd;
    bool bad = false;
    struct Regs { typename Grad::Regs g; float S[4], w[4], m[4], v[4]; };

    template <class T> __device__ __forceinline__ void init(T t, uint64_t base, const StepScalars &sc)
    {
        grad.init(t, base);
        w_in = chunk_base((const void *)t->w_in, base * 4); m_in = chunk_base((const void *)t->m_in, base * 4);
        v_in = chunk_base((const void *)t->v_in, base * 4);
        w_out = chunk_base((void *)t->w_out, base * 4); m_out = chunk_base((void *)t->m_out, base * 4);
        v_out = chunk_base((void *)t->v_out, base * 4);
        w16 = chunk_base((void *)t->w16, base * 2);
        s = sc;
        wd = t->wd;
    }
    __device__ __forceinline__ void load(Regs &x, uint32_t e) const
    {
        grad.load(x.g, e);
        ld_f32x4<Mem>(w_in, e * 4, x.w); ld_f32x4<Mem>(m_in, e * 4, x.m); ld_f32x4<Mem>(v_in, e * 4, x.v);
    }
    __device__ __forceinline__ void one(float S, float &w, float &m, float &v)
    {
        const bool nf = not_finite(S);
        bad |= nf;
        float mk = m, vk = v;
        moments<MODE>(S, w, wd, s, mk, vk);
        const float wk = __builtin_fmaf(-s.lr, direction<MODE>(w, wd, mk, vk, s), w);
        if (!(MODE & kModeGuard) || !nf) { m = mk; v = vk; w = wk; }
    }
    // compute = reduce (the sums, which settle `bad`) + update (everything else)
    __device__ __forceinline__ void reduce(Regs &x)
    {
        grad.sum(x.g, x.S);
        bad = bad || not_finite(x.S[0]) || not_finite(x.S[1]) || not_finite(x.S[2]) || not_finite(x.S[3]);
    }
    __device__ __forceinline__ void update(Regs &x)
    {
#pragma unroll
        for (int k = 0; k < 4; ++k) one(x.S[k], x.w[k], x.m[k], x.v[k]);
    }
    __device__ __forceinline__ void compute(Regs &x)
    {
        reduce(x);
        update(x);
    }
    __device__ __forceinline__ void store(const Regs &x, uint32_t e) const
    {
        st_f32x4<Mem>(m_out, e * 4, x.m); st_f32x4<Mem>(v_out, e * 4, x.v); st_f32x4<Mem>(w_out, e * 4, x.w);
        if (EMIT16) st_f16x4<Mem>(w16, e * 2, x.w);
    }
    __device__ __forceinline__ void single(uint32_t j)
    {
        float w = ld_f32(w_in, j * 4), m = ld_f32(m_in, j * 4), v = ld_f32(v_in, j * 4);
        one(grad.sum1(j), w, m, v);
        st_f32(m_out, j * 4, m); st_f32(v_out, j * 4, v); st_f32(w_out, j * 4, w);
        if (EMIT16) st_f16(w16, j * 2, w);
    }
    template <int BLOCK> __device__ __forceinline__ void end_chunk(uint32_t) {}
};

// SLICES_PLAIN: the gradient slices by plain loads, the state as Mem says (see fused_policies).
template <int R, bool GF32, class Mem, bool SLICES_PLAIN>
using AdamSlices = GradSlices<R, GF32, typename std::conditional<SLICES_PLAIN, Resident, Mem>::type>;
template <int R, int MODE, int BLOCK, bool GF32 = false, int GROUPS = 2, class Mem = Streaming, bool SLICES_PLAIN = false>
__global__ __launch_bounds__(BLOCK) void fused_adam_kernel(const DevTensor *__restrict__ tensors,
                                                           const Chunk *__restrict__ chunks, StepScalars s,
                                                           FlagScratch *__restrict__ fs, int32_t *__restrict__ flag)
{
    FlagCount<BLOCK> fc;
    fc.arrive(fs);
    const Where wh = locate(tensors, chunks, s);
    AdamOp<AdamSlices<R, GF32, Mem, SLICES_PLAIN>, MODE, true, Mem> op;
    op.init(wh.t, wh.base, s);
    sweep_and_publish<BLOCK, GROUPS>(op, wh.len, fc, fs, flag);
}

// A plan with a single tensor (the contiguous case of Table 2 and of the standalone sweep of Section 6.1.1) needs
// no table: workgroup b takes chunk b, and the descriptor travels in the kernel arguments, so the two dependent
// scalar loads (table entry, then descriptor) in front of the first vector load fall away.  ~1 us of a launch-bound
// step.
template <int R, int MODE, int BLOCK, bool GF32 = false, int GROUPS = 2, class Mem = Streaming, bool SLICES_PLAIN = false>
__global__ __launch_bounds__(BLOCK) void fused_adam_flat_kernel(DevTensor t, StepScalars s, FlagScratch *__restrict__ fs,
                                                                int32_t *__restrict__ flag)
{
    FlagCount<BLOCK> fc;
    fc.arrive(fs);
    const uint64_t base = (uint64_t)blockIdx.x * s.chunk_elems;
    const uint64_t rem = t.numel - base;
    AdamOp<AdamSlices<R, GF32, Mem, SLICES_PLAIN>, MODE, true, Mem> op;
    op.init(&t, base, s);
    sweep_and_publish<BLOCK, GROUPS>(op, rem < s.chunk_elems ? (uint32_t)rem : s.chunk_elems, fc, fs, flag);
}

// ... with its arguments in 96 bytes (see PackedAdam), in chunks of kPackedChunk.  us per eager pass, three tensors in turn,
// without / with: R = 1 4.80 / 4.22 at 1031 elements, R = 4 4.79 / 4.25 at 4099, R = 8 4.80 / 4.45 and R = 16 4.88 / 4.33 at 14000; static call, R = 2 5.38 / 4.89 at 50003;
// graph replays and shards that the device takes longer for are the same within 1 %.
constexpr uint32_t kPackedChunk = 1024;
template <int R, int MODE, int BLOCK, bool GF32, class Mem>
__global__ __launch_bounds__(BLOCK) void fused_adam_packed_kernel(PackedAdam a)
{
    FlagScratch *fs = (FlagScratch *)a.scratch;
    FlagCount<BLOCK> fc;
    fc.arrive(fs, (a.numel + (kPackedChunk - 1)) / kPackedChunk);
    DevTensor t;
    const auto at = [&](int k) { return packed_at(a, k); };
    t.w_in = (const float *)at(0); t.m_in = (const float *)at(1); t.v_in = (const float *)at(2);
    t.w_out = (float *)at(3); t.m_out = (float *)at(4); t.v_out = (float *)at(5);
    t.w16 = (uint16_t *)at(6);
#pragma unroll
    for (int r = 0; r < R; ++r) t.grad[r] = (const void *)packed_slice(a, r);
    t.wd = a.wd;
    StepScalars s;
    s.inv_div = a.inv_div;
    s.beta1 = a.beta1; s.beta2 = a.beta2; s.omb1 = 1.0 - s.beta1; s.omb2 = 1.0 - s.beta2;
    s.rc1 = a.rc1; s.rc2 = a.rc2; s.eps = a.eps; s.lr = a.lr;
    const uint32_t base = blockIdx.x * kPackedChunk, rem = a.numel - base;
    AdamOp<GradSlices<R, GF32, Mem>, MODE, true> op;
    op.init(&t, base, s);
    sweep_and_publish<BLOCK, 2>(op, rem < kPackedChunk ? rem : kPackedChunk, fc, fs, (int32_t *)packed_flag(a));
}

// The step on a list bound by HBM in single-wave workgroups, one per piece of 256 elements: kPiecesPerChunk for every entry of the table
// of 1024-element chunks, the last of a short chunk without elements.  What bounds it is DRAM, as for one tensor (kFlatPiece); the
// two dependent trips to the table and the descriptor cost less than the narrow window of addresses in flight gives.  Rule and
// figures at list_in_pieces.
constexpr uint32_t kPiecesPerChunk = 4, kPieceChunk = kFlatPiece * kPiecesPerChunk;
template <int R, int MODE, bool GF32, class Mem>
__global__ __launch_bounds__(kFlatBlock) void fused_adam_piece_kernel(const DevTensor *__restrict__ tensors, const Chunk *__restrict__ chunks,
                                                                      StepScalars s, FlagScratch *__restrict__ fs, int32_t *__restrict__ flag)
{
    uint32_t piece = blockIdx.x;         // taken here: behind the arrival's branch the compiler keeps it in a vector register
    asm volatile("" : "+s"(piece));
    FlagCount<kFlatBlock> fc;
    fc.arrive(fs);
    const ChunkEntry c = (ChunkEntry)chunks + piece / kPiecesPerChunk;
    Where wh;
    wh.index = c->index;
    wh.t = (Descriptor)tensors + c->tensor;
    all_lines(wh);
    finish_where(wh, kPieceChunk);
    const uint32_t first = piece % kPiecesPerChunk * kFlatPiece, rest = wh.len > first ? wh.len - first : 0u;
    AdamOp<GradSlices<R, GF32, Mem>, MODE, true> op;
    op.init(wh.t, wh.base + first, s);
    sweep_and_publish<kFlatBlock, 1>(op, rest < kFlatPiece ? rest : kFlatPiece, fc, fs, flag);
}

// The same step under the ordered persistent schedule (chunk_elems == BLOCK * 4 * GROUPS).
template <int R, int MODE, int BLOCK, bool GF32 = false, int GROUPS = 2>
__global__ __launch_bounds__(BLOCK) void fused_adam_ordered_kernel(const DevTensor *__restrict__ tensors,
                                                                   const Chunk *__restrict__ chunks, uint32_t nfull,
                                                                   uint32_t nchunks, uint32_t span, StepScalars s,
                                                                   WorkQueue *__restrict__ q, int32_t *__restrict__ flag)
{
    typedef AdamOp<GradSlices<R, GF32>, MODE, true> Op;
    Op a, b;
    auto bind = [&](Op &op, uint32_t entry) {
        const Where wh = locate_at(tensors, chunks, entry, s.chunk_elems);
        op.init(wh.t, wh.base, s);
        return wh;
    };
    ordered_stream<BLOCK, GROUPS>(a, b, bind, nfull, nchunks, span, q);
    leave_queue<true>(a.bad | b.bad, q, flag);
}

// Unfused pipeline, optimizer stage: the same update from the stored fp32 sum; the cast kernel emits fp16.
// In whole-step-skip mode the flag is already final here (the reduce kernel set it), so an overflowed step
// writes nothing.
template <int MODE, int BLOCK, bool SUM16 = false, class Mem = Streaming>
__global__ __launch_bounds__(BLOCK) void adam_from_sum_kernel(const DevTensor *__restrict__ tensors,
                                                              const Chunk *__restrict__ chunks, StepScalars s,
                                                              const int32_t *__restrict__ flag)
{
    if (!(MODE & kModeGuard) && *flag != 0) return;
    const Where wh = locate(tensors, chunks, s);
    AdamOp<typename std::conditional<SUM16, GradSumHalf<Mem>, GradSum<Mem>>::type, MODE, false> op;
    op.init(wh.t, wh.base, s);
    stream_chunk<BLOCK>(op, wh.len);
}

template <int MODE, int BLOCK, bool SUM16 = false>
__global__ __launch_bounds__(BLOCK) void adam_from_sum_ordered_kernel(const DevTensor *__restrict__ tensors,
                                                                      const Chunk *__restrict__ chunks, uint32_t nfull,
                                                                      uint32_t nchunks, uint32_t span, StepScalars s,
                                                                      WorkQueue *__restrict__ q, const int32_t *__restrict__ flag)
{
    if (!(MODE & kModeGuard) && *flag != 0) return;
    typedef AdamOp<typename std::conditional<SUM16, GradSumHalf<>, GradSum<>>::type, MODE, false> Op;
    Op a, b;
    auto bind = [&](Op &op, uint32_t entry) {
        const Where wh = locate_at(tensors, chunks, entry, s.chunk_elems);
        op.init(wh.t, wh.base, s);
        return wh;
    };
    ordered_stream<BLOCK, 2>(a, b, bind, nfull, nchunks, span, q);
    leave_queue<false>(false, q, nullptr);
}

// ---------------------------------------------------------------------------------------------------
// Block-wide sum of two doubles: wave butterfly, then LDS across the waves.  Same order every run.
//
// The butterfly adds to a lane's value that of the lane 32, 16, 8, 4, 2 and 1 away, in registers: gfx950's half and row swaps,
// then rotations inside a row (what a row of 16 holds after the step over 8 repeats every 8 lanes, so that a rotation by 4 meets
// the value 4 away).  Through LDS (ds_bpermute) each of the six steps waits for a trip of some 100 cycles, and the sums are what
// the rest of a small LAMB step waits for.  Same operands, same bits.  LAMB, R = 8, us per step with the butterflies, the groups'
// sums and the overflow mark through LDS and two barriers more / this: 7.31 / 6.79 at 60000 elements, 8.66 / 8.10 at 200000, 16.0 / 15.0 at
// 1.1 M, 12.2 / 11.6 at 657 K in 398 tensors; from 4 M on the same within 1 %.
// ---------------------------------------------------------------------------------------------------
template <class Swap> __device__ __forceinline__ double swap_add(double x, Swap swap)
{
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    const u32x2 lo = swap((uint32_t)__double2loint(x)), hi = swap((uint32_t)__double2hiint(x));
    return __hiloint2double((int)hi.x, (int)lo.x) + __hiloint2double((int)hi.y, (int)lo.y);
}
template <int CTRL> __device__ __forceinline__ double dpp(double x)
{
    return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(x), CTRL, 0xf, 0xf, true), __builtin_amdgcn_mov_dpp(__double2loint(x), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ double wave_sum(double x)
{
    x = swap_add(x, [](uint32_t v) { return __builtin_amdgcn_permlane32_swap(v, v, false, false); });
    x = swap_add(x, [](uint32_t v) { return __builtin_amdgcn_permlane16_swap(v, v, false, false); });
    x += dpp<0x128>(x);                  // row_ror:8
    x += dpp<0x124>(x);                  // row_ror:4
    x += dpp<0x4E>(x);                   // quad_perm:[2,3,0,1]
    x += dpp<0xB1>(x);                   // quad_perm:[1,0,3,2]
    return x;
}
// The value of one lane (the same one for the whole wave).
__device__ __forceinline__ double of_lane(double x, uint32_t lane)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), lane), __builtin_amdgcn_readlane(__double2loint(x), lane));
}

// ... and whether `any` is set anywhere in the workgroup.  AGAIN: the workgroup calls this more than once.
template <int BLOCK, bool AGAIN>
__device__ __forceinline__ void block_sum2(double &a, double &b, bool &any)
{
    constexpr int kWaves = BLOCK / 64;
    a = wave_sum(a);
    b = wave_sum(b);
    any = __builtin_amdgcn_ballot_w64(any) != 0ull;
    if (kWaves > 1) {
        __shared__ double lds[2][kWaves];
        __shared__ int some[kWaves];
        const int wave = threadIdx.x >> 6;
        if (AGAIN) __syncthreads();      // the last call's reads are over
        if ((threadIdx.x & 63) == 0) { lds[0][wave] = a; lds[1][wave] = b; some[wave] = any; }
        __syncthreads();
        a = lds[0][0];
        b = lds[1][0];
        any = some[0] != 0;
#pragma unroll
        for (int k = 1; k < kWaves; ++k) { a += lds[0][k]; b += lds[1][k]; any = any || some[k] != 0; }
    }
}

// Two sums of one launch as four words of 32 bits, each with the launch's tag (30 bits of the phase that FlagCount counts) and two
// marks next to it in one 64-bit word: whoever reads them needs no order between the words, and nothing has to be reset.
struct alignas(32) TaggedSums { unsigned long long word[4]; };
__device__ __forceinline__ unsigned long long ld_word(const unsigned long long *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Word k of the sums (sw, su), with the launch's tag and the marks.
__device__ __forceinline__ void publish(TaggedSums *p, uint32_t k, uint32_t tag, uint32_t mark, double sw, double su)
{
    const double x = k < 2 ? sw : su;
    const uint32_t half = (uint32_t)((k & 1u) ? __double2hiint(x) : __double2loint(x));
    __hip_atomic_store(&p->word[k], (unsigned long long)(tag << 2 | mark) << 32 | half, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ---------------------------------------------------------------------------------------------------
// LAMB phase 1: reduce, moments (written), and this chunk's sum(w^2), sum(u^2).
// ---------------------------------------------------------------------------------------------------
template <class Grad>
struct LambPhase1Op {
    static constexpr uint32_t kPack = kStatePack;
    typedef typename Grad::Mem Mem;
    Grad grad;
    gcbytes w_in, m_in, v_in;
    gbytes m_out, v_out;
    StepScalars s;
    float wd;
    bool bad = false;
    float sw = 0.f, su = 0.f;        // per lane: at most chunk_elems / BLOCK terms each, then double
    double *partials = nullptr;      // 2 per chunk, indexed by the chunk's position in tensor order
    struct Regs { typename Grad::Regs g; float S[4], w[4], m[4], v[4]; };

    template <class T> __device__ __forceinline__ void init(T t, uint64_t base, const StepScalars &sc)
    {
        grad.init(t, base);
        w_in = chunk_base((const void *)t->w_in, base * 4); m_in = chunk_base((const void *)t->m_in, base * 4);
        v_in = chunk_base((const void *)t->v_in, base * 4);
        m_out = chunk_base((void *)t->m_out, base * 4); v_out = chunk_base((void *)t->v_out, base * 4);
        s = sc;
        wd = t->wd;
    }
    __device__ __forceinline__ void load(Regs &x, uint32_t e) const
    {
        grad.load(x.g, e);
        ld_f32x4<typename ReadAgain<Mem>::Policy>(w_in, e * 4, x.w); ld_f32x4<Mem>(m_in, e * 4, x.m); ld_f32x4<Mem>(v_in, e * 4, x.v);
    }
    __device__ __forceinline__ void one(float S, float w, float &m, float &v)
    {
        bad |= not_finite(S);
        moments<0>(S, w, wd, s, m, v);
        const float u = direction<0>(w, wd, m, v, s);
        sw = __builtin_fmaf(w, w, sw);
        su = __builtin_fmaf(u, u, su);
    }
    __device__ __forceinline__ void reduce(Regs &x)
    {
        grad.sum(x.g, x.S);
        bad = bad || not_finite(x.S[0]) || not_finite(x.S[1]) || not_finite(x.S[2]) || not_finite(x.S[3]);
    }
    __device__ __forceinline__ void update(Regs &x)
    {
#pragma unroll
        for (int k = 0; k < 4; ++k) one(x.S[k], x.w[k], x.m[k], x.v[k]);
    }
    __device__ __forceinline__ void compute(Regs &x)
    {
        reduce(x);
        update(x);
    }
    __device__ __forceinline__ void store(const Regs &x, uint32_t e) const
    {
        st_f32x4<Mem>(m_out, e * 4, x.m); st_f32x4<Mem>(v_out, e * 4, x.v);
    }
    __device__ __forceinline__ void single(uint32_t j)
    {
        const float w = ld_f32(w_in, j * 4);
        float m = ld_f32(m_in, j * 4), v = ld_f32(v_in, j * 4);
        one(grad.sum1(j), w, m, v);
        st_f32(m_out, j * 4, m); st_f32(v_out, j * 4, v);
    }
    // The chunk's two partial sums: lanes in fp32, then wave butterfly and LDS in double, always in the same order.
    template <int BLOCK, bool AGAIN = true> __device__ __forceinline__ void end_chunk(uint32_t slot)
    {
        double dw = sw, du = su;
        bool unused = false;
        block_sum2<BLOCK, AGAIN>(dw, du, unused);
        if (threadIdx.x == 0) {
            partials[2 * (uint64_t)slot] = dw;
            partials[2 * (uint64_t)slot + 1] = du;
        }
        sw = su = 0.f;
    }
};

// Half of LAMB's second level inside its first sweep (see lamb_tallies): as a launch of its own, one workgroup per tensor, it leaves the
// device idle for 4.6 us at 5 to 24 M elements.  Here a workgroup publishes its chunk's sums as tagged words and counts itself in
// its group: the chunks that one wave of that launch adds up, those with the same (index / 64) % 16.  Whoever completes the group
// adds them up; the second sweep adds up its tensor's 16 groups.  Where every tensor is one group, which is all of its sums, so does the
// first of the two phase calls (lamb_phase1_sums).  Same additions in the same order as tensor_sums, so the same bits.
//   * The words carry the launch's tag, so that the count needs no order behind them: the last one to count looks until all
//     the words are there.  All of them have been issued by then; nobody waits for a workgroup that has not run.
//   * The counts only grow.  Every launch adds a power of two to each, because the group's first chunk adds for those that are
//     missing, and who gets to a multiple of it is the last one.  Nothing is reset, and calls that overlap on one plan, which the
//     interface forbids, leave the counts as they should be.  The bound ends a look for words that another launch has overwritten:
//     the sums are then incomplete, and the wave reports an overflow, through the state word, since the flag may not be cleared yet.
constexpr int kNormBlock = 1024;         // lanes in whose order a tensor's chunks are added up (see tensor_sums)
constexpr uint32_t kNormGroups = kNormBlock / 64;
constexpr int kTallyBlock = 128;         // threads of the workgroups that do this
struct LambTally {
    struct alignas(16) Sums { double w, u; };
    struct alignas(128) Count { uint32_t chunks; };
    TaggedSums *chunk;                   // by slot; nullptr: plain partial sums, which lamb_norms_kernel adds up
    Count *count;                        // by DevTensor::first_group + which group of the tensor
    Sums *group;                         // as well; nullptr: every tensor is one group, and its sums go to `sums`
    Sums *sums;                          // by tensor
};

// One look of a wave at n sums, lane by lane and `rows` of them, 1024 apart, per lane: adds them up as tensor_sums does if all are this launch's.
template <int ROWS>
__device__ __forceinline__ bool tally_look(const TaggedSums *p, uint32_t first, uint32_t n, uint32_t tag, double (&sw)[4], double (&su)[4])
{
    unsigned long long x[ROWS][4];
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
#pragma unroll
        for (int k = 0; k < 4; ++k) x[r][k] = first + r * kNormBlock < n ? ld_word(&p[first + r * kNormBlock].word[k]) : (unsigned long long)(tag << 2) << 32;
    bool here = true;
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
#pragma unroll
        for (int k = 0; k < 4; ++k) here = here && (uint32_t)(x[r][k] >> 34) == tag;
    if (__builtin_amdgcn_ballot_w64(!here) != 0ull) return false;
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        sw[r] += __hiloint2double((int)(uint32_t)x[r][1], (int)(uint32_t)x[r][0]);
        su[r] += __hiloint2double((int)(uint32_t)x[r][3], (int)(uint32_t)x[r][2]);
    }
    return true;
}

// A chunk's sums (sw, su), by one wave of its workgroup.  True if it completes its group.
__device__ __forceinline__ bool tally_chunk(const LambTally &ty, const Where &wh, uint32_t tag, double sw, double su)
{
    const uint32_t lane = threadIdx.x & 63u, n = wh.t->num_chunks, g = wh.index / 64u % kNormGroups;
    if (lane < 4u) publish(ty.chunk + wh.slot, lane, tag, 0u, sw, su);
    // `rows` of 1024 chunks, 64 of each in every group, and what is left
    const uint32_t rows = n / kNormBlock, left = n % kNormBlock;
    const uint32_t members = rows * 64u + (left > g * 64u ? (left - g * 64u < 64u ? left - g * 64u : 64u) : 0u);
    uint32_t most = 64u, was = 0u;
    while (most < members) most *= 2u;
    const uint32_t add = wh.index == g * 64u ? most - members + 1u : 1u;
    if (lane == 0u) was = __hip_atomic_fetch_add(&ty.count[wh.t->first_group + g].chunks, add, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return (((uint32_t)__builtin_amdgcn_readfirstlane((int)was) + add) & (most - 1u)) == 0u;
}

// ... and then this, for all of the group.  False (for the whole wave): words were lost.
__device__ __forceinline__ bool tally_group(const LambTally &ty, const Where &wh, uint32_t tag)
{
    const uint32_t lane = threadIdx.x & 63u, n = wh.t->num_chunks, g = wh.index / 64u % kNormGroups;
    const TaggedSums *all = ty.chunk + (wh.slot - wh.index);
    double a[4] = {0.0, 0.0, 0.0, 0.0}, b[4] = {0.0, 0.0, 0.0, 0.0};
    uint32_t looks = 0;
    bool lost = false;
    for (uint32_t c = g * 64u; c < n; c += 4u * kNormBlock)
        while (!(c + kNormBlock < n ? tally_look<4>(all, c + lane, n, tag, a, b) : tally_look<1>(all, c + lane, n, tag, a, b)))
            if ((lost = ++looks > kMeetingBound)) break;
    const double tw = wave_sum((a[0] + a[1]) + (a[2] + a[3])), tu = wave_sum((b[0] + b[1]) + (b[2] + b[3]));
    if (lane == 0u) (ty.group != nullptr ? ty.group[wh.t->first_group + g] : ty.sums[wh.tensor]) = LambTally::Sums{tw, tu};
    return !lost;
}

// The sums of a tensor of n chunks from those of its groups, for the whole wave.
__device__ __forceinline__ void tally_sums(const LambTally::Sums *group, uint32_t n, double &sw, double &su)
{
    const uint32_t lane = threadIdx.x & 63u, groups = n < (uint32_t)kNormBlock ? (n + 63u) / 64u : kNormGroups;
    LambTally::Sums mine{0.0, 0.0};
    if (lane < groups) mine = group[lane];
    sw = of_lane(mine.w, 0);
    su = of_lane(mine.u, 0);
#pragma unroll
    for (uint32_t k = 1; k < kNormGroups; ++k) { sw += of_lane(mine.w, k); su += of_lane(mine.u, k); }
}

// One chunk of the first sweep whose sums go into the tally.  One wave publishes them and counts before it stores its part of the chunk
// (as well off with the stores first: 20.96 / 20.99 us at 2.5 M elements, R = 2).
template <int BLOCK, class Op>
__device__ __forceinline__ void sweep_and_tally(Op &op, const Where &wh, const LambTally &ty, FlagCount<BLOCK> &fc, FlagScratch *fs, int32_t *flag)
{
    typedef Sweep<BLOCK, 2, Op> S;
    const bool whole = wh.len >= Op::kPack && wh.len <= 2 * S::kGroup;
    S sw;
    if (whole) {
        sw.load(op, wh.len);
        __builtin_amdgcn_sched_barrier(0);
        fc.slot_level(fs);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int g = 0; g < 2; ++g) op.reduce(sw.x[g]);
        fc.top_level(fs, flag);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int g = 0; g < 2; ++g)
            if (S::mine(g, wh.len)) op.update(sw.x[g]);
        ragged_end(op, wh.len);
    } else {
        stream_chunk<BLOCK, Op, 2>(op, wh.len);
        fc.slot_level(fs);
        fc.top_level(fs, flag);
    }
    double dw = op.sw, du = op.su;
    bool unused = false, last = false;
    block_sum2<BLOCK, false>(dw, du, unused);
    const uint32_t tag = (uint32_t)__builtin_amdgcn_readfirstlane((int)fc.tag()) & 0x3fffffffu;
    if (threadIdx.x >= BLOCK - 64u) last = tally_chunk(ty, wh, tag, dw, du);
    __builtin_amdgcn_sched_barrier(0);
    if (whole) {
#pragma unroll
        for (int g = 0; g < 2; ++g)
            if (S::mine(g, wh.len)) op.store(sw.x[g], S::first(g));
    }
    __builtin_amdgcn_sched_barrier(0);
    fc.finish(op.bad, fs, flag);
    if (last && !tally_group(ty, wh, tag) && fc.counting_lane()) fc.report(fs, flag);
}

template <class Grad, bool RAISE, int BLOCK>
__device__ __forceinline__ void lamb_phase1_body(const DevTensor *__restrict__ tensors, const Chunk *__restrict__ chunks,
                                                 const StepScalars &s, double *__restrict__ partials, const LambTally &tally,
                                                 FlagScratch *__restrict__ fs, int32_t *__restrict__ flag)
{
    FlagCount<BLOCK> fc;
    if (RAISE) fc.arrive(fs);
    const Where wh = locate(tensors, chunks, s);
    LambPhase1Op<Grad> op;
    op.init(wh.t, wh.base, s);
    op.partials = partials;
    if constexpr (RAISE && BLOCK == kTallyBlock) {
        if (tally.chunk != nullptr) return sweep_and_tally<BLOCK>(op, wh, tally, fc, fs, flag);
    }
    if (RAISE) {
        sweep_and_publish<BLOCK, 2>(op, wh.len, fc, fs, flag);
    } else {
        stream_chunk<BLOCK>(op, wh.len);
    }
    op.template end_chunk<BLOCK, false>(wh.slot);
}

template <class Grad, bool RAISE, int BLOCK>
__device__ __forceinline__ void lamb_phase1_ordered_body(const DevTensor *__restrict__ tensors, const Chunk *__restrict__ chunks,
                                                         uint32_t nfull, uint32_t nchunks, uint32_t span, const StepScalars &s,
                                                         double *__restrict__ partials, WorkQueue *__restrict__ q,
                                                         int32_t *__restrict__ flag)
{
    typedef LambPhase1Op<Grad> Op;
    Op a, b;
    a.partials = b.partials = partials;
    auto bind = [&](Op &op, uint32_t entry) {
        const Where wh = locate_at(tensors, chunks, entry, s.chunk_elems);
        op.init(wh.t, wh.base, s);
        return wh;
    };
    ordered_stream<BLOCK, 2>(a, b, bind, nfull, nchunks, span, q);
    leave_queue<RAISE>(a.bad | b.bad, q, flag);
}

template <int R, int BLOCK, bool GF32 = false>
__global__ __launch_bounds__(BLOCK) void lamb_phase1_ordered_kernel(const DevTensor *__restrict__ tensors,
                                                                    const Chunk *__restrict__ chunks, uint32_t nfull,
                                                                    uint32_t nchunks, uint32_t span, StepScalars s,
                                                                    double *__restrict__ partials, WorkQueue *__restrict__ q,
                                                                    int32_t *__restrict__ flag)
{
    lamb_phase1_ordered_body<GradSlices<R, GF32>, true, BLOCK>(tensors, chunks, nfull, nchunks, span, s, partials, q, flag);
}

template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void lamb_phase1_from_sum_ordered_kernel(const DevTensor *__restrict__ tensors,
                                                                             const Chunk *__restrict__ chunks, uint32_t nfull,
                                                                             uint32_t nchunks, uint32_t span, StepScalars s,
                                                                             double *__restrict__ partials,
                                                                             WorkQueue *__restrict__ q)
{
    lamb_phase1_ordered_body<GradSum<>, false, BLOCK>(tensors, chunks, nfull, nchunks, span, s, partials, q, nullptr);
}

template <int R, int BLOCK, bool GF32 = false, class Mem = Streaming>
__global__ __launch_bounds__(BLOCK) void lamb_phase1_kernel(const DevTensor *__restrict__ tensors,
                                                            const Chunk *__restrict__ chunks, StepScalars s,
                                                            double *__restrict__ partials, LambTally tally,
                                                            FlagScratch *__restrict__ fs, int32_t *__restrict__ flag)
{
    lamb_phase1_body<GradSlices<R, GF32, Mem>, true, BLOCK>(tensors, chunks, s, partials, tally, fs, flag);
}

template <int BLOCK, class Mem = Streaming>
__global__ __launch_bounds__(BLOCK) void lamb_phase1_from_sum_kernel(const DevTensor *__restrict__ tensors,
                                                                     const Chunk *__restrict__ chunks, StepScalars s,
                                                                     double *__restrict__ partials)
{
    lamb_phase1_body<GradSum<Mem>, false, BLOCK>(tensors, chunks, s, partials, LambTally{}, nullptr, nullptr);
}

// LAMB second level: a tensor's chunk partials are added in a fixed order, so the result does not change between runs
// or between the launch shapes below.  The order is that of 1024 lanes: lane v adds the chunks v, v + 1024, ... into four
// independent strided partial sums, the lanes of each 64-wide wave are added by a butterfly and the 16 wave totals one
// after the other.  A workgroup of BLOCK < 1024 threads plays 1024 / BLOCK lanes per thread: its wave w stands for the
// waves w, w + BLOCK / 64, ... of the wide one, so every addition has the same operands.
template <int BLOCK>
__device__ __forceinline__ void tensor_sums(const double *__restrict__ p, uint32_t n, double &sa, double &sb)
{
    constexpr int kRealWaves = BLOCK / 64, kWaves = kNormBlock / 64, kPlayed = kNormBlock / BLOCK;
    static_assert(kNormBlock % BLOCK == 0 && BLOCK % 64 == 0, "a workgroup plays whole waves");
    __shared__ double lds[2][kWaves];
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    __syncthreads();                     // a caller may use the function twice: the last call's reads are over
    if (n <= (uint32_t)kNormBlock) {
        // At most one chunk per lane: the lane's four strided sums are that chunk's value and zeros, i.e. the value
        // itself, so all loads can be issued at once (a lane that plays eight would otherwise wait eight times).
        double ta[kPlayed], tb[kPlayed];
#pragma unroll
        for (int j = 0; j < kPlayed; ++j) {
            const uint32_t c = (wave + j * kRealWaves) * 64 + lane;
            ta[j] = c < n ? p[2 * (uint64_t)c] : 0.0;
            tb[j] = c < n ? p[2 * (uint64_t)c + 1] : 0.0;
        }
#pragma unroll
        for (int j = 0; j < kPlayed; ++j) {
            const uint32_t played_wave = wave + j * kRealWaves;
            if (played_wave * 64 < n) { ta[j] = wave_sum(ta[j]); tb[j] = wave_sum(tb[j]); }
            if (lane == 0) { lds[0][played_wave] = ta[j]; lds[1][played_wave] = tb[j]; }
        }
    } else
#pragma unroll
    for (int j = 0; j < kPlayed; ++j) {
        const uint32_t played_wave = wave + j * kRealWaves;
        double ta = 0.0, tb = 0.0;
        if (played_wave * 64 < n) {      // a wave without chunks adds up zeros: the same +0.0, without the work
            double a[4] = {0.0, 0.0, 0.0, 0.0}, b[4] = {0.0, 0.0, 0.0, 0.0};
            uint32_t c = played_wave * 64 + lane;
            for (; c + 3 * kNormBlock < n; c += 4 * kNormBlock) {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    a[k] += p[2 * (uint64_t)(c + k * kNormBlock)];
                    b[k] += p[2 * (uint64_t)(c + k * kNormBlock) + 1];
                }
            }
            for (int k = 0; c < n; c += kNormBlock, ++k) {
                a[k] += p[2 * (uint64_t)c];
                b[k] += p[2 * (uint64_t)c + 1];
            }
            ta = wave_sum((a[0] + a[1]) + (a[2] + a[3]));
            tb = wave_sum((b[0] + b[1]) + (b[2] + b[3]));
        }
        if (lane == 0) { lds[0][played_wave] = ta; lds[1][played_wave] = tb; }
    }
    __syncthreads();
    sa = lds[0][0];
    sb = lds[1][0];
#pragma unroll
    for (int k = 1; k < kWaves; ++k) { sa += lds[0][k]; sb += lds[1][k]; }
}

// One workgroup per tensor.
[[maybe_unused]] static __global__ __launch_bounds__(kNormBlock) void lamb_norms_kernel(const DevTensor *__restrict__ tensors,
                                                                const double *__restrict__ partials,
                                                                double *__restrict__ sums)
{
    const Descriptor t = (Descriptor)tensors + blockIdx.x;
    double sa, sb;
    tensor_sums<kNormBlock>(partials + 2 * (uint64_t)t->first_chunk, t->num_chunks, sa, sb);
    if (threadIdx.x == 0) {
        sums[2 * (uint64_t)blockIdx.x] = sa;
        sums[2 * (uint64_t)blockIdx.x + 1] = sb;
    }
}

// LAMB phase 2: the same u from the stored moments, scaled by the tensor's ratio.  EMIT16 = false in the
// unfused pipeline, where a separate cast kernel writes the fp16 copy.
template <bool EMIT16, class Mem = Streaming>
struct LambPhase2Op {
    static constexpr uint32_t kPack = kStatePack;
    gcbytes w_in, m_new, v_new;
    gbytes w_out, w16;
    StepScalars s;
    float wd, step;
    struct Regs { float w[4], m[4], v[4]; };

    // Everything but the ratio: the loads need none.
    template <class T> __device__ __forceinline__ void init(T t, uint64_t base, const StepScalars &sc)
    {
        w_in = chunk_base((const void *)t->w_in, base * 4);
        m_new = chunk_base((const void *)t->m_out, base * 4); v_new = chunk_base((const void *)t->v_out, base * 4);
        w_out = chunk_base((void *)t->w_out, base * 4); w16 = chunk_base((void *)t->w16, base * 2);
        s = sc;
        wd = t->wd;
    }
    // ... formed from the tensor's sums of w^2 and u^2.
    __device__ __forceinline__ void scale(double sw, double su)
    {
        const float ratio = (sw > 0.0 && su > 0.0) ? (float)(__builtin_sqrt(sw) / __builtin_sqrt(su)) : 1.0f;
        step = s.lr * ratio;
    }
    __device__ __forceinline__ void load(Regs &x, uint32_t e) const
    {
        ld_f32x4<Mem>(w_in, e * 4, x.w); ld_f32x4<Mem>(m_new, e * 4, x.m); ld_f32x4<Mem>(v_new, e * 4, x.v);
    }
    __device__ __forceinline__ float one(float w, float m, float v) const
    {
        return __builtin_fmaf(-step, direction<0>(w, wd, m, v, s), w);
    }
    __device__ __forceinline__ void update(Regs &x) const
    {
#pragma unroll
        for (int k = 0; k < 4; ++k) x.w[k] = one(x.w[k], x.m[k], x.v[k]);
    }
    __device__ __forceinline__ void compute(Regs &x) const { update(x); }
    __device__ __forceinline__ void store(const Regs &x, uint32_t e) const
    {
        st_f32x4<Mem>(w_out, e * 4, x.w);
        if (EMIT16) st_f16x4<Mem>(w16, e * 2, x.w);
    }
    __device__ __forceinline__ void single(uint32_t j)
    {
        const float wn = one(ld_f32(w_in, j * 4), ld_f32(m_new, j * 4), ld_f32(v_new, j * 4));
        st_f32(w_out, j * 4, wn);
        if (EMIT16) st_f16(w16, j * 2, wn);
    }
    template <int BLOCK> __device__ __forceinline__ void end_chunk(uint32_t) {}
};

template <bool EMIT16, int BLOCK, class Mem = Streaming, bool TALLIED = false>
__global__ __launch_bounds__(BLOCK) void lamb_phase2_kernel(const DevTensor *__restrict__ tensors,
                                                            const Chunk *__restrict__ chunks, StepScalars s,
                                                            double *__restrict__ sums, const LambTally::Sums *__restrict__ group,
                                                            const int32_t *__restrict__ flag)
{
    const Where wh = locate<true>(tensors, chunks, s);
    LambPhase2Op<EMIT16, Mem> op;
    op.init(wh.t, wh.base, s);
    sweep_when_ready<BLOCK, 2>(op, wh.len, [&] {
        const int32_t overflowed = *flag;
        double sw, su;
        if (TALLIED) {
            tally_sums(group + wh.t->first_group, wh.t->num_chunks, sw, su);
            if (wh.index == 0 && threadIdx.x == 0) {
                sums[2 * (uint64_t)wh.tensor] = sw;
                sums[2 * (uint64_t)wh.tensor + 1] = su;
            }
        } else {
            sw = sums[2 * (uint64_t)wh.tensor];
            su = sums[2 * (uint64_t)wh.tensor + 1];
        }
        if (overflowed != 0) return false;    // whole-step skip: w and w16 stay as they were
        op.scale(sw, su);
        return true;
    });
}

// Phase 2 of a plan whose tensors have few chunks each, with the second level folded in: every workgroup adds up the
// partials of its own tensor (the same additions in the same order as lamb_norms_kernel, so the same bits), which
// costs 16 bytes per chunk of the tensor from the L2 and saves a launch.  The workgroup of a tensor's first chunk
// also stores the sums, so that they can be read back as after the separate kernel.
template <bool EMIT16, int BLOCK, class Mem = Streaming>
__global__ __launch_bounds__(BLOCK) void lamb_phase2_with_norms_kernel(const DevTensor *__restrict__ tensors,
                                                                       const Chunk *__restrict__ chunks, StepScalars s,
                                                                       const double *__restrict__ partials,
                                                                       double *__restrict__ sums,
                                                                       const int32_t *__restrict__ flag)
{
    const Where wh = locate<true>(tensors, chunks, s);
    LambPhase2Op<EMIT16, Mem> op;
    op.init(wh.t, wh.base, s);
    sweep_when_ready<BLOCK, 2>(op, wh.len, [&] {
        const int32_t overflowed = *flag;
        double sw, su;
        tensor_sums<BLOCK>(partials + 2 * (uint64_t)wh.t->first_chunk, wh.t->num_chunks, sw, su);
        if (wh.index == 0 && threadIdx.x == 0) {
            sums[2 * (uint64_t)wh.tensor] = sw;
            sums[2 * (uint64_t)wh.tensor + 1] = su;
        }
        if (overflowed != 0) return false;       // whole-step skip: w and w16 stay as they were
        op.scale(sw, su);
        return true;
    });
}

// LAMB in one launch, for shards of at most kMeetingMostChunks chunks of 1024 elements (see lamb_meets).  Such a step is mostly latency: as
// two launches it pays for the end of a kernel, the start of the next and a second trip to memory between the partial sums
// and their use.  Here every workgroup keeps its chunk in registers, publishes its sums and waits for those of the others.
// Same sums in the same order and the same update from the same values, so the same bits as in two launches.
// Two launches / one, us per step, one tensor, R = 8, graph replay: 6.8 / 5.4 at 1024 elements, 7.6 / 5.7 at 10007, 8.0 / 6.5
// at 30000, 8.7 / 7.5 at 65000; eager calls, which also save the host a launch, 7.5-9.2 / 5.1-5.9 up to 10007 elements.
//
//   * A workgroup publishes its two sums as four words of 32 bits, each with the launch's tag next to it in one 64-bit
//     word, so that a reader needs no order between the words and nothing has to be reset: words of other launches carry
//     other tags (30 bits of the phase that FlagCount counts, which wrap).  A bit beside the tag tells whether the workgroup
//     saw an inf/NaN: with the sums a wave learns whether the step is to be skipped, before it writes w.  (One chunk's words
//     lie together: by word, 64 chunks in four lines, a wave looks at fewer lines but the chunks' stores meet in them: 5.7 ->
//     6.4 us at 10007 elements.)
//   * Up to kMeetingChunks chunks lane i of every wave polls chunk i of its tensor, and the first word of chunk i of the shard.
//     Beyond that (GROUPED) too many waves would look at too many lines (8.5 us at 128 chunks, 10.0 at 254, where two launches
//     take 9.0 to 9.6): the second wave of every 64th workgroup of a tensor adds up 64 chunks and publishes the group's sums,
//     and every wave polls groups.  They are published in kGroupCopies copies, one for the workgroups of each XCD, so that not
//     all of them read the same lines, and polls are 0.4 us apart (at 1024 chunks 16.8 us with none between them, 16.1 with
//     0.4, 15.5 with 1.3, which costs 0.6 at 100).
//   * No wait depends on how many of the workgroups the device holds at a time (several steps on as many streams, other
//     kernels in the way, a stream that may use one compute unit).  A workgroup publishes before it waits.  The wave that
//     FlagCount finds to be the last arrival of the launch knows that all workgroups have started, so all of them will
//     publish.  Any other wave, the one that adds up a group included, gives up in the end: it moves the word `outcome` to
//     (tag, ABANDONED) and leaves, its part of w unwritten.  Half of the workgroups do so after `limit` looks, some tens of
//     microseconds, and so make room for those that have not started; the others stay kMeetingPatience times as long.
//   * The last arrival, once it has all it needs, exchanges the word for (tag, CLOSED).  If ABANDONED was there it puts that
//     back, and it and whoever else is there share the work of those that have left: they take the shard's chunks from a counter in the same
//     word and compute their w again, from all chunks' sums and the step's inputs, which a LAMB step never overwrites.
//     Whoever wrote its own part meanwhile wrote the same values.  A wave learns that some have left from the word, which it looks
//     at every kMeetingGlance looks, or from another bit beside the tags (a workgroup that leaves sets its own): one that started late,
//     and finds everything published at once, helps as well.  One that started late and does not find it stays for a few looks only.
//     A wave that finds CLOSED when it would give up knows that everything has been published and looks on.
//   * One tensor, R = 8, us for a step beside a kernel that leaves 4 of the 256 compute units free for another 160 us / 960 us, two
//     launches / one: 157 / 172 and 957 / 970 at 128 chunks; 158 / 177 and 957 / 976 at 256.
//   * Calls that overlap on one plan, which the interface forbids, mix the arrivals and words of two launches; kMeetingBound
//     ends the waits that would then have no end, and a wave that took itself for the last arrival sets the overflow flag.
struct LambMeeting {
    FlagScratch flag;                                                // what the other kernels use
    FlagScratch::Line outcome;
    typedef TaggedSums Sums;
    Sums chunk[kMeetingMostChunks], group[kGroupCopies][kMeetingGroups];
};
// `outcome`: two bits of state, the tag, and from kTicket on the next chunk to be computed again.
constexpr unsigned long long kAbandoned = 1ull, kClosed = 2ull, kTicket = 1ull << 32;
__device__ __forceinline__ bool marks(unsigned long long word, unsigned long long mark) { return (word & (kTicket - 1ull)) == mark; }

// Marks beside the tag: a workgroup saw an inf/NaN; one has left.
constexpr uint32_t kMarkBad = 1u, kMarkGone = 2u;

// One look of a wave at n <= 64 sums from `p` on (lane i gets the i-th, the others zeros) and at the marks of those and of
// the m <= 64 from `q` on (`mark`: all of them together).  True (for the whole wave) if all of them are this launch's.
__device__ __forceinline__ bool look(const TaggedSums *p, uint32_t n, const TaggedSums *q, uint32_t m, uint32_t tag, double &sw,
                                     double &su, uint32_t &mark)
{
    const uint32_t lane = threadIdx.x & 63u;
    unsigned long long x[4] = {}, y = 0ull;
    if (lane < n) {
#pragma unroll
        for (int k = 0; k < 4; ++k) x[k] = ld_word(&p[lane].word[k]);
    }
    if (lane < m) y = ld_word(q[lane].word);
    bool here = lane >= m || (uint32_t)(y >> 34) == tag;
#pragma unroll
    for (int k = 0; k < 4; ++k) here = here && (lane >= n || (uint32_t)(x[k] >> 34) == tag);
    if (__builtin_amdgcn_ballot_w64(!here) != 0ull) return false;
    const uint32_t seen = (uint32_t)((x[0] | y) >> 32);
    mark = (__builtin_amdgcn_ballot_w64((seen & kMarkBad) != 0u) != 0ull ? kMarkBad : 0u) |
           (__builtin_amdgcn_ballot_w64((seen & kMarkGone) != 0u) != 0ull ? kMarkGone : 0u);
    sw = __hiloint2double((int)(uint32_t)x[1], (int)(uint32_t)x[0]);
    su = __hiloint2double((int)(uint32_t)x[3], (int)(uint32_t)x[2]);
    return true;
}

// Whether some wave of this launch has left (for the whole wave).
__device__ __forceinline__ bool abandoned(const LambMeeting *mt, unsigned long long mark)
{
    const bool yes = (threadIdx.x & 63u) == 0u && marks(ld_word(&mt->outcome.word), mark);
    return __builtin_amdgcn_ballot_w64(yes) != 0ull;
}

// A wave has waited long enough.  True: `outcome` says that some have left, and it may leave.
__device__ __forceinline__ bool give_up(LambMeeting *mt, unsigned long long left, unsigned long long closed)
{
    unsigned long long cur = 0ull;
    if ((threadIdx.x & 63u) == 0u) {
        cur = ld_word(&mt->outcome.word);
        while (!marks(cur, left) && !marks(cur, closed))
            if (__hip_atomic_compare_exchange_strong(&mt->outcome.word, &cur, left, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) cur = left;
    }
    return __builtin_amdgcn_ballot_w64((threadIdx.x & 63u) == 0u && marks(cur, left)) != 0ull;
}

// A wave's waiting in one launch.
struct Wait {
    enum Next { kLook, kLeave, kHelp };
    unsigned long long left, closed;     // what `outcome` reads when a wave has left, when none will
    uint32_t polls = 0, most;            // looks in vain so far, and how many before this wave gives up
    bool last, stays, sure = false;      // the launch's last arrival; one of those that stay; everything has been published
    __device__ __forceinline__ Wait(uint32_t tag, uint32_t limit, bool last_) : last(last_)
    {
        left = (unsigned long long)tag << 2 | kAbandoned;
        closed = (unsigned long long)tag << 2 | kClosed;
        stays = meeting_stays(blockIdx.x);
        most = !stays ? limit : limit > kMeetingBound / kMeetingPatience ? kMeetingBound : limit * kMeetingPatience;
    }
    // A look has been in vain.
    __device__ __forceinline__ Next again(LambMeeting *mt)
    {
        if (++polls > kMeetingBound) return kLeave;
        if (!last && !sure && polls > most) {
            if (give_up(mt, left, closed)) return kLeave;
            sure = true;
        }
        if ((polls & (kMeetingGlance - 1u)) != 0u || sure || !abandoned(mt, left)) return kLook;
        if (!stays || polls == kMeetingGlance) most = polls + kMeetingLinger;
        return kHelp;
    }
};

template <class Grad, bool GROUPED, int BLOCK, int WAVES>
__global__ __launch_bounds__(BLOCK, WAVES) void lamb_one_launch_kernel(const DevTensor *__restrict__ per_chunk, StepScalars s,
                                                                double *__restrict__ sums, LambMeeting *__restrict__ mt,
                                                                int32_t *__restrict__ flag, uint32_t limit, uint32_t total_groups)
{
    typedef typename Grad::Mem Mem;
    typedef LambPhase1Op<Grad> Op;
    typedef Sweep<BLOCK, 2, Op> S;
    static_assert(BLOCK == 128, "the second wave leads a group while the first one publishes");
    FlagCount<BLOCK> fc;
    fc.arrive(&mt->flag);
    const Where wh = locate(per_chunk, nullptr, s);
    Op op;
    op.init(wh.t, wh.base, s);
    // The whole packs and the ragged end's elements, all loads together.  (Lanes without one load the chunk's first.)
    S sw;
    const bool packs = wh.len >= Op::kPack, rest = threadIdx.x < (wh.len & (Op::kPack - 1));
    const uint32_t j = (wh.len & ~(Op::kPack - 1u)) + threadIdx.x;
    const uint32_t j1 = rest ? j : 0u;
    typename Grad::One g1;
    op.grad.load1(g1, j1);
    float w1 = ld_f32(op.w_in, j1 * 4), m1 = ld_f32(op.m_in, j1 * 4), v1 = ld_f32(op.v_in, j1 * 4);
    if (packs) sw.load(op, wh.len);
    __builtin_amdgcn_sched_barrier(0);
    fc.slot_level(&mt->flag);
    __builtin_amdgcn_sched_barrier(0);
    if (packs) {
#pragma unroll
        for (int g = 0; g < 2; ++g) op.reduce(sw.x[g]);
    }
    fc.top_level(&mt->flag, flag);
#pragma unroll
    for (int g = 0; g < 2; ++g)
        if (S::mine(g, wh.len)) op.update(sw.x[g]);
    if (rest) op.one(Grad::sum1(g1), w1, m1, v1);
    double dw = op.sw, du = op.su;
    bool block_bad = op.bad;
    block_sum2<BLOCK, false>(dw, du, block_bad);
    const uint32_t tag = (uint32_t)__builtin_amdgcn_readfirstlane((int)fc.tag()) & 0x3fffffffu;
    if (threadIdx.x < 4) publish(&mt->chunk[wh.slot], threadIdx.x, tag, block_bad ? kMarkBad : 0u, dw, du);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int g = 0; g < 2; ++g)
        if (S::mine(g, wh.len)) op.store(sw.x[g], S::first(g));
    if (rest) { st_f32(op.m_out, j * 4, m1); st_f32(op.v_out, j * 4, v1); }

    const uint32_t lane = threadIdx.x & 63u, total = gridDim.x, n = wh.t->num_chunks;
    Wait wait(tag, limit, __builtin_amdgcn_ballot_w64(fc.launch_last) != 0ull);   // uniform: this wave is the last arrival
    Wait::Next next = Wait::kLook;
    double tw = 0.0, tu = 0.0;
    uint32_t mark = 0u;
    if (GROUPED && (wh.index & 63u) == 0u && threadIdx.x >= 64u) {                // this wave adds up a group of chunks
        const uint32_t members = n - wh.index < 64u ? n - wh.index : 64u;
        while (!look(&mt->chunk[wh.slot], members, nullptr, 0u, tag, tw, tu, mark)) {
            __builtin_amdgcn_s_sleep(1);
            if ((next = wait.again(mt)) != Wait::kLook) break;
        }
        if (next == Wait::kLook) {
            tw = wave_sum(tw);
            tu = wave_sum(tu);
            if (lane < 4u * kGroupCopies) publish(&mt->group[lane >> 2][wh.t->first_group + (wh.index >> 6)], lane & 3u, tag, mark, tw, tu);
        }
    }
    // What this wave waits for: its tensor's sums, by chunk or by group, and everybody's marks.
    const TaggedSums *all = GROUPED ? mt->group[blockIdx.x % kGroupCopies] : mt->chunk;
    const uint32_t first = GROUPED ? wh.t->first_group : wh.t->first_chunk, count = GROUPED ? (n + 63u) >> 6 : n;
    const uint32_t everybody = GROUPED ? total_groups : total, others = count == everybody ? 0u : everybody;
    while (next == Wait::kLook && !look(all + first, count, all, others, tag, tw, tu, mark)) {
        __builtin_amdgcn_s_sleep(GROUPED ? 16 : 1);
        next = wait.again(mt);
    }
    LambPhase2Op<true, Mem> p2;
    const auto finish_pack = [&](const typename Op::Regs &x, uint32_t e) {
        typename LambPhase2Op<true, Mem>::Regs y;
#pragma unroll
        for (int k = 0; k < 4; ++k) { y.w[k] = x.w[k]; y.m[k] = x.m[k]; y.v[k] = x.v[k]; }
        p2.update(y);
        p2.store(y, e);
    };
    const auto finish_one = [&](float w, float m, float v, uint32_t e) {
        const float wn = p2.one(w, m, v);
        st_f32(p2.w_out, e * 4, wn);
        st_f16(p2.w16, e * 2, wn);
    };
    unsigned long long was = 0ull;
    if (next == Wait::kLook) {
        if (wait.last && lane == 0u) was = __hip_atomic_exchange(&mt->outcome.word, wait.closed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        // as tensor_sums adds up to 1024 chunks: 64 at a time by a butterfly, and those one after the other
        if (GROUPED) {
            const double gw = tw, gu = tu;
            tw = tu = 0.0;
            for (uint32_t g = 0; g < count; ++g) { tw += of_lane(gw, g); tu += of_lane(gu, g); }
        } else {
            tw = wave_sum(tw);
            tu = wave_sum(tu);
        }
        p2.init(wh.t, wh.base, s);
        p2.scale(tw, tu);
        if (wh.index == 0 && threadIdx.x == 0) { sums[2 * (uint64_t)wh.tensor] = tw; sums[2 * (uint64_t)wh.tensor + 1] = tu; }
        if (!(mark & kMarkBad)) {        // whole-step skip: w and w16 stay as they were
#pragma unroll
            for (int g = 0; g < 2; ++g)
                if (S::mine(g, wh.len)) finish_pack(sw.x[g], S::first(g));
            if (rest) finish_one(w1, m1, v1, j);
        }
    }
    fc.finish(op.bad, &mt->flag, flag);
    const auto lost = [&]() {            // only where calls have overlapped: no w that this wave vouches for
        if (wait.last && lane == 0u) __hip_atomic_store(flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    if (next == Wait::kLeave) {
        if (lane == 0u) publish(&mt->chunk[wh.slot], 0u, tag, kMarkGone | (block_bad ? kMarkBad : 0u), dw, du);
        return lost();
    }
    if (next == Wait::kLook) {
        if (wait.last) {
            if (__builtin_amdgcn_ballot_w64(lane == 0u && marks(was, wait.left)) == 0ull) return;        // nobody has left, and nobody will
            if (lane == 0u) __hip_atomic_exchange(&mt->outcome.word, was, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else if ((wait.polls < kMeetingGlance && !(mark & kMarkGone)) || !abandoned(mt, wait.left)) {
            return;
        }
    }
    // Some waves have left: the shard's chunks once more, one after the other from the counter, by the waves that are here.
    // First all the chunks' marks, which also tell that all their sums are there.
    bool skip = false;
    for (uint32_t c = 0; c < total;) {
        if (look(&mt->chunk[c], total - c < 64u ? total - c : 64u, nullptr, 0u, tag, tw, tu, mark)) {
            skip = skip || (mark & kMarkBad) != 0u;
            c += 64u;
            continue;
        }
        __builtin_amdgcn_s_sleep(1);
        if (++wait.polls > (wait.last ? kMeetingBound : wait.most)) return lost();
    }
    uint32_t summed = ~0u;               // the tensor whose sums p2's scale is from
    while (true) {
        unsigned long long ticket = 0ull;
        if (lane == 0u) ticket = __hip_atomic_fetch_add(&mt->outcome.word, kTicket, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (__builtin_amdgcn_ballot_w64(lane == 0u && marks(ticket, wait.left)) == 0ull) return lost();
        const uint32_t c = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(ticket >> 32));
        if (c >= total) return;
        Where at;
        at.t = (Descriptor)per_chunk + c;
        at.index = at.t->chunk_index;
        finish_where(at, s.chunk_elems);
        p2.init(at.t, at.base, s);
        if (at.t->tensor != summed) {
            summed = at.t->tensor;
            double cw = 0.0, cu = 0.0;
            for (uint32_t g = 0; g < at.t->num_chunks; g += 64u) {
                const uint32_t members = at.t->num_chunks - g < 64u ? at.t->num_chunks - g : 64u;
                if (!look(&mt->chunk[c - at.index + g], members, nullptr, 0u, tag, tw, tu, mark)) return lost();
                cw += wave_sum(tw);
                cu += wave_sum(tu);
            }
            tw = cw;
            tu = cu;
        }
        p2.scale(tw, tu);
        if (at.index == 0 && lane == 0u) { sums[2 * (uint64_t)at.t->tensor] = tw; sums[2 * (uint64_t)at.t->tensor + 1] = tu; }
        if (skip) continue;
        Op again;
        again.init(at.t, at.base, s);
        for (uint32_t e = lane * Op::kPack; e + Op::kPack <= at.len; e += 2u * 64u * Op::kPack) {
            const uint32_t e2 = e + 64u * Op::kPack;
            const bool two = e2 + Op::kPack <= at.len;
            again.load(sw.x[0], e);
            again.load(sw.x[1], two ? e2 : e);
            __builtin_amdgcn_sched_barrier(0);
            again.compute(sw.x[0]);
            finish_pack(sw.x[0], e);
            if (two) { again.compute(sw.x[1]); finish_pack(sw.x[1], e2); }
        }
        const uint32_t r = (at.len & ~(Op::kPack - 1u)) + lane;
        if (r < at.len) {
            float w = ld_f32(again.w_in, r * 4), m = ld_f32(again.m_in, r * 4), v = ld_f32(again.v_in, r * 4);
            again.one(again.grad.sum1(r), w, m, v);
            finish_one(w, m, v, r);
        }
    }
}

template <bool EMIT16, int BLOCK>
__global__ __launch_bounds__(BLOCK) void lamb_phase2_ordered_kernel(const DevTensor *__restrict__ tensors,
                                                                    const Chunk *__restrict__ chunks, uint32_t nfull,
                                                                    uint32_t nchunks, uint32_t span, StepScalars s,
                                                                    const double *__restrict__ sums, WorkQueue *__restrict__ q,
                                                                    const int32_t *__restrict__ flag)
{
    if (*flag != 0) return;
    typedef LambPhase2Op<EMIT16> Op;
    Op a, b;
    auto bind = [&](Op &op, uint32_t entry) {
        const Where wh = locate_at(tensors, chunks, entry, s.chunk_elems);
        op.init(wh.t, wh.base, s);
        op.scale(sums[2 * (uint64_t)wh.tensor], sums[2 * (uint64_t)wh.tensor + 1]);
        return wh;
    };
    ordered_stream<BLOCK, 2>(a, b, bind, nfull, nchunks, span, q);
    leave_queue<false>(false, q, nullptr);
}

// ---------------------------------------------------------------------------------------------------
// Unfused pipeline pieces: reduce to an fp32 buffer, and the fp32 -> fp16 cast.
// ---------------------------------------------------------------------------------------------------
template <int R, bool GF32, class Mem = Streaming>
struct ReduceOp {
    static constexpr uint32_t kPack = kStatePack;
    GradSlices<R, GF32, Mem> grad;
    gbytes gsum;
    bool bad = false;
    struct Regs { typename GradSlices<R, GF32, Mem>::Regs g; float S[4]; };
    template <class T> __device__ __forceinline__ void init(T t, uint64_t base)
    {
        grad.init(t, base);
        gsum = chunk_base((void *)t->gsum, base * 4);
    }
    __device__ __forceinline__ void load(Regs &x, uint32_t e) const { grad.load(x.g, e); }
    __device__ __forceinline__ void compute(Regs &x)
    {
        grad.sum(x.g, x.S);
        bad = bad || not_finite(x.S[0]) || not_finite(x.S[1]) || not_finite(x.S[2]) || not_finite(x.S[3]);
    }
    __device__ __forceinline__ void store(const Regs &x, uint32_t e) const { st_f32x4<Mem>(gsum, e * 4, x.S); }
    __device__ __forceinline__ void single(uint32_t j)
    {
        const float S = grad.sum1(j);
        bad |= not_finite(S);
        st_f32(gsum, j * 4, S);
    }
    template <int BLOCK> __device__ __forceinline__ void end_chunk(uint32_t) {}
};

template <int R, int BLOCK, bool GF32 = false, class Mem = Streaming>
__global__ __launch_bounds__(BLOCK) void reduce_kernel(const DevTensor *__restrict__ tensors,
                                                       const Chunk *__restrict__ chunks, StepScalars s,
                                                       FlagScratch *__restrict__ fs, int32_t *__restrict__ flag)
{
    FlagCount<BLOCK> fc;
    fc.arrive(fs);
    const Where wh = locate(tensors, chunks, s);
    ReduceOp<R, GF32, Mem> op;
    op.init(wh.t, wh.base);
    stream_chunk<BLOCK>(op, wh.len);
    fc.settle(op.bad, fs, flag);
}

template <int R, int BLOCK, bool GF32 = false>
__global__ __launch_bounds__(BLOCK) void reduce_ordered_kernel(const DevTensor *__restrict__ tensors,
                                                               const Chunk *__restrict__ chunks, uint32_t nfull,
                                                               uint32_t nchunks, uint32_t span, StepScalars s, WorkQueue *__restrict__ q,
                                                               int32_t *__restrict__ flag)
{
    typedef ReduceOp<R, GF32> Op;
    Op a, b;
    auto bind = [&](Op &op, uint32_t entry) {
        const Where wh = locate_at(tensors, chunks, entry, s.chunk_elems);
        op.init(wh.t, wh.base);
        return wh;
    };
    ordered_stream<BLOCK, 2>(a, b, bind, nfull, nchunks, span, q);
    leave_queue<true>(a.bad | b.bad, q, flag);
}

// The reduce stage of the fp16 all-reduce baseline: the sum of the R fp16 slices leaves as fp16.  The slices are
// added in double (exact for up to 16 fp16 values) and rounded to fp32, then to fp16, so that the stored value is
// fp16(fp32(sum)) whatever the order of the additions.  The flag is decided on the fp16 value: a finite sum beyond
// 65504 comes back as inf, as it would from an fp16 collective.
template <int R, class Mem = Streaming>
struct ReduceHalfOp {
    static constexpr uint32_t kPack = kStatePack;
    GradSlices<R, false, Mem> grad;
    gbytes gsum;
    bool bad = false;
    struct Regs { typename GradSlices<R, false, Mem>::Regs g; float S[4]; };
    template <class T> __device__ __forceinline__ void init(T t, uint64_t base)
    {
        grad.init(t, base);
        gsum = chunk_base((void *)t->gsum, base * 2);
    }
    __device__ __forceinline__ void load(Regs &x, uint32_t e) const { grad.load(x.g, e); }
    static __device__ __forceinline__ float through_half(double s, bool &bad)
    {
        const float h = (float)to_half((float)s);
        bad = bad || not_finite(h);
        return h;
    }
    __device__ __forceinline__ void compute(Regs &x)
    {
        double a = (double)(float)x.g.g[0].x, b = (double)(float)x.g.g[0].y, c = (double)(float)x.g.g[0].z, d = (double)(float)x.g.g[0].w;
#pragma unroll
        for (int r = 1; r < R; ++r) {
            a += (double)(float)x.g.g[r].x; b += (double)(float)x.g.g[r].y; c += (double)(float)x.g.g[r].z; d += (double)(float)x.g.g[r].w;
        }
        x.S[0] = through_half(a, bad); x.S[1] = through_half(b, bad); x.S[2] = through_half(c, bad); x.S[3] = through_half(d, bad);
    }
    __device__ __forceinline__ void store(const Regs &x, uint32_t e) const { st_f16x4<Mem>(gsum, e * 2, x.S); }
    __device__ __forceinline__ void single(uint32_t j)
    {
        double S = (double)ld_f16(grad.g[0], j * 2);
#pragma unroll
        for (int r = 1; r < R; ++r) S += (double)ld_f16(grad.g[r], j * 2);
        st_f16(gsum, j * 2, through_half(S, bad));
    }
    template <int BLOCK> __device__ __forceinline__ void end_chunk(uint32_t) {}
};

template <int R, int BLOCK, class Mem = Streaming>
__global__ __launch_bounds__(BLOCK) void reduce_half_kernel(const DevTensor *__restrict__ tensors,
                                                            const Chunk *__restrict__ chunks, StepScalars s,
                                                            FlagScratch *__restrict__ fs, int32_t *__restrict__ flag)
{
    FlagCount<BLOCK> fc;
    fc.arrive(fs);
    const Where wh = locate(tensors, chunks, s);
    ReduceHalfOp<R, Mem> op;
    op.init(wh.t, wh.base);
    stream_chunk<BLOCK>(op, wh.len);
    fc.settle(op.bad, fs, flag);
}

template <int R, int BLOCK>
__global__ __launch_bounds__(BLOCK) void reduce_half_ordered_kernel(const DevTensor *__restrict__ tensors,
                                                                    const Chunk *__restrict__ chunks, uint32_t nfull,
                                                                    uint32_t nchunks, uint32_t span, StepScalars s, WorkQueue *__restrict__ q,
                                                                    int32_t *__restrict__ flag)
{
    typedef ReduceHalfOp<R> Op;
    Op a, b;
    auto bind = [&](Op &op, uint32_t entry) {
        const Where wh = locate_at(tensors, chunks, entry, s.chunk_elems);
        op.init(wh.t, wh.base);
        return wh;
    };
    ordered_stream<BLOCK, 2>(a, b, bind, nfull, nchunks, span, q);
    leave_queue<true>(a.bad | b.bad, q, flag);
}

template <class Mem = Streaming>
struct CastOp {
    static constexpr uint32_t kPack = kStatePack;
    gcbytes w_new;
    gbytes w16;
    struct Regs { float w[4]; };
    template <class T> __device__ __forceinline__ void init(T t, uint64_t base)
    {
        w_new = chunk_base((const void *)t->w_out, base * 4);
        w16 = chunk_base((void *)t->w16, base * 2);
    }
    __device__ __forceinline__ void load(Regs &x, uint32_t e) const { ld_f32x4<Mem>(w_new, e * 4, x.w); }
    __device__ __forceinline__ void compute(Regs &) {}
    __device__ __forceinline__ void store(const Regs &x, uint32_t e) const { st_f16x4<Mem>(w16, e * 2, x.w); }
    __device__ __forceinline__ void single(uint32_t j) { st_f16(w16, j * 2, ld_f32(w_new, j * 4)); }
    template <int BLOCK> __device__ __forceinline__ void end_chunk(uint32_t) {}
};

// fp32 master weights -> fp16 copy.  `guarded`: leave w16 alone on overflow (whole-step skip).
template <int BLOCK, class Mem = Streaming>
__global__ __launch_bounds__(BLOCK) void cast_kernel(const DevTensor *__restrict__ tensors,
                                                     const Chunk *__restrict__ chunks, StepScalars s,
                                                     const int32_t *__restrict__ flag, int guarded)
{
    if (guarded && *flag != 0) return;
    const Where wh = locate(tensors, chunks, s);
    CastOp<Mem> op;
    op.init(wh.t, wh.base);
    stream_chunk<BLOCK>(op, wh.len);
}

template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void cast_ordered_kernel(const DevTensor *__restrict__ tensors,
                                                             const Chunk *__restrict__ chunks, uint32_t nfull,
                                                             uint32_t nchunks, uint32_t span, StepScalars s, WorkQueue *__restrict__ q,
                                                             const int32_t *__restrict__ flag, int guarded)
{
    if (guarded && *flag != 0) return;
    CastOp<> a, b;
    auto bind = [&](CastOp<> &op, uint32_t entry) {
        const Where wh = locate_at(tensors, chunks, entry, s.chunk_elems);
        op.init(wh.t, wh.base);
        return wh;
    };
    ordered_stream<BLOCK, 2>(a, b, bind, nfull, nchunks, span, q);
    leave_queue<false>(false, q, nullptr);
}

// ---------------------------------------------------------------------------------------------------
// Model-parallel epilogue (Fig. 3 with the schedule of Fig. 5, program 3) on one rank's slice:
//     out = Dropout(partial_0 + ... + partial_{R-1} + bias, p) + residual,  every tensor fp16.
// All streams are fp16, so a lane owns 8 consecutive elements and every access is 16 bytes (1 KiB per wave
// instruction).  2R + 4 bytes per element.  The dropout mask is a counter-based generator of the global element
// index (Philox4x32 with 10 rounds: counter = index / 4, key = seed, word index % 4), so that it does not depend on
// how the tensor is sliced or chunked; an element is kept iff its word >= floor(p 2^32).
// ---------------------------------------------------------------------------------------------------
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

struct EpilogueArgs {
    uint64_t numel;           // elements of this slice
    uint64_t first;           // global index of the slice's first element (multiple of 8)
    uint32_t hidden;          // H: the bias column of global element i is i % H (multiple of 8)
    uint32_t threshold;       // floor(p 2^32)
    uint32_t key0, key1;      // seed, low and high half
    float scale;              // 1 / (1 - p)
    const uint16_t *partial[CC_MAX_R];
    const uint16_t *bias;
    const uint16_t *residual;
    uint16_t *out;
    float *sum;               // unfused pipeline only: fp32 reduced partial outputs
    uint32_t runs;            // fused kernel: take the pieces in runs per XCD (piece_in_runs)
};

__device__ __forceinline__ void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0, uint32_t k1,
                                              uint32_t (&out)[4])
{
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        const uint32_t hi0 = __umulhi(0xD2511F53u, c0), lo0 = 0xD2511F53u * c0;
        const uint32_t hi1 = __umulhi(0xCD9E8D57u, c2), lo1 = 0xCD9E8D57u * c2;
        c0 = hi1 ^ c1 ^ k0;
        c1 = lo1;
        c2 = hi0 ^ c3 ^ k1;
        c3 = lo0;
        k0 += 0x9E3779B9u;      // the key schedule; the bump after the last round is unused
        k1 += 0xBB67AE85u;
    }
    out[0] = c0; out[1] = c1; out[2] = c2; out[3] = c3;
}

// The pointwise part for one element whose reduced sum is x_sum (fp32).
__device__ __forceinline__ float epilogue_value(float x_sum, float bias, float residual, bool keep, float scale)
{
    const float x = x_sum + bias;
    return (keep ? x * scale : 0.0f) + residual;
}

// The epilogue's accesses: non-temporal loads, stores written through (see cc_fused_epilogue).
__device__ __forceinline__ f16x8 ld_f16x8(gcbytes b, uint32_t off) { return __builtin_nontemporal_load((const CCF_GLOBAL f16x8 *)(b + off)); }
__device__ __forceinline__ void st_f16x8(gbytes b, uint32_t off, f16x8 x) { st_f32x4<WriteThrough>(b, off, __builtin_bit_cast(f32x4, x)); }

// Common part of the fused kernel and of the unfused pipeline's pointwise kernel: mask, bias column, output.
struct EpilogueTail {
    gcbytes res, bias;
    gbytes out;
    uint64_t gbase;           // global index of the chunk's first element
    uint32_t col_base;        // bias column of the chunk's first element
    uint32_t hidden, threshold, k0, k1;
    float scale;
    __device__ __forceinline__ void init(const EpilogueArgs &a, uint64_t base)
    {
        res = chunk_base((const void *)a.residual, base * 2);
        bias = (gcbytes)a.bias;
        out = chunk_base((void *)a.out, base * 2);
        gbase = a.first + base;
        col_base = (uint32_t)(gbase % a.hidden);
        hidden = a.hidden; threshold = a.threshold; k0 = a.key0; k1 = a.key1; scale = a.scale;
    }
    // words of the Philox block that holds global elements 4q .. 4q+3, q = (gbase + e) / 4
    __device__ __forceinline__ void words(uint32_t e, uint32_t (&w)[4]) const
    {
        const uint64_t block = (gbase + e) >> 2;
        philox4x32_10((uint32_t)block, (uint32_t)(block >> 32), 0u, 0u, k0, k1, w);
    }
    __device__ __forceinline__ uint32_t column(uint32_t e) const { return (col_base + e) % hidden; }
    __device__ __forceinline__ void single(uint32_t j, float x_sum) const
    {
        uint32_t w[4];
        words(j, w);
        const bool keep = w[(gbase + j) & 3] >= threshold;
        st_f16(out, j * 2, epilogue_value(x_sum, ld_f16(bias, column(j) * 2), ld_f16(res, j * 2), keep, scale));
    }
};

template <int R>
struct FusedEpilogueOp {
    static constexpr uint32_t kPack = 8;
    gcbytes part[R];
    EpilogueTail t;
    struct Regs { f16x8 p[R]; f16x8 r; f16x8 b; uint32_t e; };
    __device__ __forceinline__ void init(const EpilogueArgs &a, uint64_t base)
    {
#pragma unroll
        for (int r = 0; r < R; ++r) part[r] = chunk_base((const void *)a.partial[r], base * 2);
        t.init(a, base);
    }
    __device__ __forceinline__ void load(Regs &x, uint32_t e) const
    {
#pragma unroll
        for (int r = 0; r < R; ++r) x.p[r] = ld_f16x8(part[r], e * 2);
        x.r = ld_f16x8(t.res, e * 2);
        x.b = *(const CCF_GLOBAL f16x8 *)(t.bias + t.column(e) * 2);     // 8 columns never wrap: H and e are multiples of 8
        x.e = e;
    }
    __device__ __forceinline__ void compute(Regs &x)
    {
        uint32_t w[8];
        uint32_t lo[4], hi[4];
        t.words(x.e, lo);
        t.words(x.e + 4, hi);
#pragma unroll
        for (int k = 0; k < 4; ++k) { w[k] = lo[k]; w[4 + k] = hi[k]; }
        f16x8 o;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            float sum = (float)x.p[0][k];
#pragma unroll
            for (int r = 1; r < R; ++r) sum += (float)x.p[r][k];
            o[k] = to_half(epilogue_value(sum, (float)x.b[k], (float)x.r[k], w[k] >= t.threshold, t.scale));
        }
        x.r = o;
    }
    __device__ __forceinline__ void store(const Regs &x, uint32_t e) const { st_f16x8(t.out, e * 2, x.r); }
    __device__ __forceinline__ void single(uint32_t j)
    {
        float sum = ld_f16(part[0], j * 2);
#pragma unroll
        for (int r = 1; r < R; ++r) sum += ld_f16(part[r], j * 2);
        t.single(j, sum);
    }
};

// Bound by reading HBM (2R + 2 of its 2R + 4 bytes per element); the mask generator's integer arithmetic hides behind
// that (the kernel without it takes as long).  Single-wave workgroups of one group per lane come and go independently
// and are the fastest shape at every R and size (two groups per lane: 0-9 % slower, 256 and 512 threads 1-5 %); what
// they gain beyond that comes from the addresses in flight, see cc_fused_epilogue.
constexpr int kEpilogueFusedBlock = 64;
constexpr uint32_t kEpiloguePiece = kEpilogueFusedBlock * 8;
template <int R>
__device__ __forceinline__ void fused_epilogue_piece(const EpilogueArgs &a, uint32_t piece)
{
    const uint64_t base = (uint64_t)piece * kEpiloguePiece;
    const uint64_t rem = a.numel - base;
    FusedEpilogueOp<R> op;
    op.init(a, base);
    stream_chunk<kEpilogueFusedBlock, FusedEpilogueOp<R>, 1>(op, rem < kEpiloguePiece ? (uint32_t)rem : kEpiloguePiece);
}
template <int R>
__global__ __launch_bounds__(kEpilogueFusedBlock) void fused_epilogue_kernel(EpilogueArgs a)
{
    fused_epilogue_piece<R>(a, a.runs ? piece_in_runs(blockIdx.x, gridDim.x) : blockIdx.x);
}
// ... with its arguments in 96 bytes.  us per eager call, three sets of buffers in turn, without / with:
// 40304 elements, R = 1 4.08 / 3.52, R = 8 4.25 / 3.89; 1 M, R = 8 5.05 / 4.60.
template <int R>
__global__ __launch_bounds__(kEpilogueFusedBlock) void fused_epilogue_packed_kernel(PackedEpilogue<R> p)
{
    EpilogueArgs a;
    a.numel = p.numel; a.first = p.first; a.hidden = p.hidden; a.threshold = p.threshold; a.key0 = p.key0; a.key1 = p.key1; a.scale = p.scale;
    const auto at = [&](int k) { return unpack_address(p.base, p.at[k]); };
#pragma unroll
    for (int r = 0; r < R; ++r) a.partial[r] = (const uint16_t *)at(r);
    a.bias = (const uint16_t *)at(R); a.residual = (const uint16_t *)at(R + 1); a.out = (uint16_t *)at(R + 2);
    fused_epilogue_piece<R>(a, blockIdx.x);
}

// Unfused pipeline: reduce the R partial outputs into an fp32 buffer (a lane owns 4 elements, so that the fp32
// stores of a wave are contiguous), then the pointwise kernel on that buffer.
template <int R>
struct EpilogueReduceOp {
    static constexpr uint32_t kPack = 4;
    gcbytes part[R];
    gbytes sum;
    struct Regs { f16x4 p[R]; float S[4]; };
    __device__ __forceinline__ void init(const EpilogueArgs &a, uint64_t base)
    {
#pragma unroll
        for (int r = 0; r < R; ++r) part[r] = chunk_base((const void *)a.partial[r], base * 2);
        sum = chunk_base((void *)a.sum, base * 4);
    }
    __device__ __forceinline__ void load(Regs &x, uint32_t e) const
    {
#pragma unroll
        for (int r = 0; r < R; ++r) x.p[r] = ld_f16x4<Streaming>(part[r], e * 2);
    }
    __device__ __forceinline__ void compute(Regs &x)
    {
        x.S[0] = (float)x.p[0].x; x.S[1] = (float)x.p[0].y; x.S[2] = (float)x.p[0].z; x.S[3] = (float)x.p[0].w;
#pragma unroll
        for (int r = 1; r < R; ++r) { x.S[0] += (float)x.p[r].x; x.S[1] += (float)x.p[r].y; x.S[2] += (float)x.p[r].z; x.S[3] += (float)x.p[r].w; }
    }
    __device__ __forceinline__ void store(const Regs &x, uint32_t e) const { st_f32x4<Streaming>(sum, e * 4, x.S); }
    __device__ __forceinline__ void single(uint32_t j)
    {
        float S = ld_f16(part[0], j * 2);
#pragma unroll
        for (int r = 1; r < R; ++r) S += ld_f16(part[r], j * 2);
        st_f32(sum, j * 4, S);
    }
};

struct EpiloguePointwiseOp {
    static constexpr uint32_t kPack = 4;
    gcbytes sum;
    EpilogueTail t;
    struct Regs { float S[4]; f16x4 r; f16x4 b; uint32_t e; };
    __device__ __forceinline__ void init(const EpilogueArgs &a, uint64_t base)
    {
        sum = chunk_base((const void *)a.sum, base * 4);
        t.init(a, base);
    }
    __device__ __forceinline__ void load(Regs &x, uint32_t e) const
    {
        ld_f32x4<Streaming>(sum, e * 4, x.S);
        x.r = ld_f16x4<Streaming>(t.res, e * 2);
        x.b = *(const CCF_GLOBAL f16x4 *)(t.bias + t.column(e) * 2);
        x.e = e;
    }
    __device__ __forceinline__ void compute(Regs &x)
    {
        uint32_t w[4];
        t.words(x.e, w);
        const float b[4] = {(float)x.b.x, (float)x.b.y, (float)x.b.z, (float)x.b.w};
        const float r[4] = {(float)x.r.x, (float)x.r.y, (float)x.r.z, (float)x.r.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) x.S[k] = epilogue_value(x.S[k], b[k], r[k], w[k] >= t.threshold, t.scale);
    }
    __device__ __forceinline__ void store(const Regs &x, uint32_t e) const { st_f16x4<Streaming>(t.out, e * 2, x.S); }
    __device__ __forceinline__ void single(uint32_t j) { t.single(j, ld_f32(sum, j * 4)); }
};

template <int R, int BLOCK>
__global__ __launch_bounds__(BLOCK) void epilogue_reduce_kernel(EpilogueArgs a)
{
    constexpr uint32_t kChunk = BLOCK * 4 * 2;
    const uint64_t base = (uint64_t)blockIdx.x * kChunk;
    const uint64_t rem = a.numel - base;
    EpilogueReduceOp<R> op;
    op.init(a, base);
    stream_chunk<BLOCK>(op, rem < kChunk ? (uint32_t)rem : kChunk);
}

template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void epilogue_pointwise_kernel(EpilogueArgs a)
{
    constexpr uint32_t kChunk = BLOCK * 4 * 2;
    const uint64_t base = (uint64_t)blockIdx.x * kChunk;
    const uint64_t rem = a.numel - base;
    EpiloguePointwiseOp op;
    op.init(a, base);
    stream_chunk<BLOCK>(op, rem < kChunk ? (uint32_t)rem : kChunk);
}

// Measurement aid: the memory pattern of the small-shard fused Adam step (one workgroup of BLOCK per BLOCK x 8 elements
// of one flat tensor, R fp16 + 3 fp32 streams in, 3 fp32 + 1 fp16 streams out) with parts taken away, to see where a
// launch-bound step's time goes.  WHAT 0: nothing (an empty workgroup), 1: the loads only, 2: the stores only,
// 3: loads and stores without the update arithmetic and without the flag.
template <int R, int WHAT, int BLOCK, class Mem>
__global__ __launch_bounds__(BLOCK) void pattern_probe_kernel(DevTensor t, StepScalars s, int32_t *__restrict__ sink)
{
    if (WHAT == 0) return;
    typedef AdamOp<GradSlices<R, false, Mem>, 0, true> Op;
    constexpr uint32_t kGroup = BLOCK * Op::kPack;
    Op op;
    op.init(&t, (uint64_t)blockIdx.x * (2 * kGroup), s);
    const uint32_t lane_e = threadIdx.x * Op::kPack;
    typename Op::Regs x[2];
#pragma unroll
    for (int g = 0; g < 2; ++g) {
        if (WHAT != 2) {
            op.load(x[g], g * kGroup + lane_e);
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k) { x[g].w[k] = (float)threadIdx.x; x[g].m[k] = (float)blockIdx.x; x[g].v[k] = 1.f; }
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    if (WHAT == 1) {
        float acc = 0.f;
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            op.grad.sum(x[g].g, x[g].S);
#pragma unroll
            for (int k = 0; k < 4; ++k) acc += x[g].S[k] + x[g].w[k] + x[g].m[k] + x[g].v[k];
        }
        if (acc == 123.456f) *sink = 1;              // keeps the loads alive; never true for the probe's data
        return;
    }
#pragma unroll
    for (int g = 0; g < 2; ++g) {
        if (WHAT == 3) {
            op.grad.sum(x[g].g, x[g].S);
#pragma unroll
            for (int k = 0; k < 4; ++k) x[g].w[k] += x[g].S[k];
        }
        op.store(x[g], g * kGroup + lane_e);
    }
}

// Plain streaming copy, 16 bytes per lane, four accesses in flight per lane.
constexpr int kCopyBlock = 256;
[[maybe_unused]] static __global__ __launch_bounds__(kCopyBlock) void copy_kernel(u32x4 *__restrict__ dst, const u32x4 *__restrict__ src,
                                                          uint64_t n16)
{
    const uint64_t base = (uint64_t)blockIdx.x * (kCopyBlock * 4) + threadIdx.x;
    u32x4 x[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint64_t i = base + (uint64_t)k * kCopyBlock;
        if (i < n16) x[k] = __builtin_nontemporal_load(src + i);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint64_t i = base + (uint64_t)k * kCopyBlock;
        if (i < n16) __builtin_nontemporal_store(x[k], dst + i);
    }
}

}  // namespace ccf
