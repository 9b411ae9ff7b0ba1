// Kernel arguments of the calls that wait for the host, in 96 bytes.  No HIP in here: the host can run it as well.
//
// A launch whose arguments take more than 96 bytes costs the host 0.55 us more, and a loop of launches 0.65 us, whether they are 104 or
// 560 bytes (same kernel, 88 / 96 / 104 / 152 / 304 bytes: 2.64 / 2.70 / 3.18 / 3.20 / 3.20 us).  A kernel that asks for its grid's size has
// 256 bytes of hidden ones.  So addresses travel as multiples of 16 bytes above the lowest one (4 bytes each, 64 GiB apart at most),
// the gradient slices as the first one's and the distance between them, and the number of workgroups follows from the sizes.
// What does not fit goes by the kernels that take everything as it is.
#pragma once

#include <stdint.h>

#include "piece_order.hpp"

namespace ccf {

// The lowest of the addresses, down to a multiple of 16.
inline uint64_t packed_base(const uint64_t *address, int n)
{
    uint64_t base = address[0];
    for (int k = 1; k < n; ++k)
        if (address[k] < base) base = address[k];
    return base & ~(uint64_t)15;
}
inline bool pack_address(uint64_t address, uint64_t base, uint32_t *out)
{
    const uint64_t d = address - base;
    if (d % 16 != 0 || d / 16 > 0xffffffffull) return false;
    *out = (uint32_t)(d / 16);
    return true;
}
CCF_ANYWHERE uint64_t unpack_address(uint64_t base, uint32_t at) { return base + (uint64_t)at * 16; }

// The distance from each of R addresses to the next, if it is one.
inline bool pack_stride(const uint64_t *address, int R, int32_t *out)
{
    const int64_t apart = R > 1 ? (int64_t)(address[1] - address[0]) : 0;
    if (apart % 16 != 0 || apart / 16 < INT32_MIN || apart / 16 > INT32_MAX) return false;
    for (int r = 2; r < R; ++r)
        if ((int64_t)(address[r] - address[r - 1]) != apart) return false;
    *out = (int32_t)(apart / 16);
    return true;
}

// The fused Adam step on one tensor.
struct PackedAdam {
    uint64_t base_flag, scratch;         // the base, and in its low bits where the flag lies in its 16 bytes; the flag's counting words
    double inv_div;
    uint32_t at[8];                      // w_in, m_in, v_in, w_out, m_out, v_out, w16, first slice
    int32_t stride;                      // from slice to slice, in 16 bytes
    uint32_t flag;
    uint32_t numel;
    float wd, beta1, beta2, rc1, rc2, eps, lr;
};
static_assert(sizeof(PackedAdam) == 96, "one more costs half a microsecond");

constexpr uint64_t kPackedMaxElems = 0xffffffffull - 0xffffu;         // rounded up to whole workgroups it still fits 32 bits
// Everything that is an address; false if it does not fit.
inline bool pack_adam(const uint64_t (&address)[8], const uint64_t *grad, int R, uint64_t flag, uint64_t scratch, uint64_t numel, PackedAdam *a)
{
    if (numel > kPackedMaxElems) return false;
    uint64_t all[9];
    for (int k = 0; k < 8; ++k) all[k] = address[k];
    all[8] = flag & ~(uint64_t)15;
    const uint64_t base = packed_base(all, 9);
    a->base_flag = base | (flag & 15);
    a->scratch = scratch;
    a->numel = (uint32_t)numel;
    for (int k = 0; k < 8; ++k)
        if (!pack_address(address[k], base, &a->at[k])) return false;
    if (!pack_address(all[8], base, &a->flag)) return false;
    return pack_stride(grad, R, &a->stride);
}
CCF_ANYWHERE uint64_t packed_at(const PackedAdam &a, int k) { return unpack_address(a.base_flag & ~(uint64_t)15, a.at[k]); }
CCF_ANYWHERE uint64_t packed_slice(const PackedAdam &a, int r) { return packed_at(a, 7) + (uint64_t)((int64_t)a.stride * 16 * r); }
CCF_ANYWHERE uint64_t packed_flag(const PackedAdam &a) { return unpack_address(a.base_flag, a.flag); }

// The fused epilogue on up to nine partial outputs.
constexpr int kPackedEpilogueMaxR = 9;
template <int R> struct PackedEpilogue {
    uint64_t base, numel, first;
    uint32_t hidden, threshold, key0, key1;
    float scale;
    uint32_t at[R + 3];                  // partial outputs, bias, residual, out
};
static_assert(sizeof(PackedEpilogue<kPackedEpilogueMaxR>) <= 96, "one more costs half a microsecond");

inline bool pack_epilogue(const uint64_t *address, int n, uint64_t *base, uint32_t *at)
{
    *base = packed_base(address, n);
    for (int k = 0; k < n; ++k)
        if (!pack_address(address[k], *base, &at[k])) return false;
    return true;
}

}  // namespace ccf
