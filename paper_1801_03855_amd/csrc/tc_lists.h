// Device access to the per-layer tensors of a tensor list, shared by the
// kernels that read or write lists.
#pragma once

#include "tc_internal.h"

namespace tc {
namespace {

typedef unsigned int u2 __attribute__((ext_vector_type(2)));
typedef unsigned int u4 __attribute__((ext_vector_type(4)));

// Bytes [sh, sh + 16) of the 32-byte little-endian concatenation lo:hi.
__device__ __forceinline__ u4 funnel(u4 lo, u4 hi, uint32_t sh) {
    const uint32_t w[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
    const uint32_t d4 = sh >> 2, b = sh & 3;
    uint32_t t[5];
#pragma unroll
    for (int q = 0; q < 5; ++q)
        t[q] = d4 == 0 ? w[q] : d4 == 1 ? w[q + 1] : d4 == 2 ? w[q + 2] : w[q + 3];
    return u4{__builtin_amdgcn_alignbyte(t[1], t[0], b), __builtin_amdgcn_alignbyte(t[2], t[1], b),
              __builtin_amdgcn_alignbyte(t[3], t[2], b), __builtin_amdgcn_alignbyte(t[4], t[3], b)};
}

// SB source bytes at address S (SB = 16 or 8; S a multiple of the element
// size): one load, non-temporal when S is SB-aligned, else one unaligned
// (cacheable) access.  Measured on MI355X against reading the two aligned
// 16-byte granules that hold the bytes and funnel-shifting them: the
// 10,000-tensor bfloat16 pack at K = 16 +5.7% (5.21 -> 5.51 TB/s), the
// pipelined step on that group +2.6%.
template <int SB>
__device__ __forceinline__ u4 load_bytes(uintptr_t S) {
    if ((S & (SB - 1)) == 0) {
        if constexpr (SB == 16) return gld_nt<u4>(S);
        const u2 w = gld_nt<u2>(S);
        return u4{w.x, w.y, 0u, 0u};
    }
    if constexpr (SB == 16) return gld_u<u4>(S);
    const u2 w = gld_u<u2>(S);
    return u4{w.x, w.y, 0u, 0u};
}

// Elements e .. e + U - 1 of one copy where they lie in several tensors, `seg`
// to at most `last`: f(k, address) for the first `cnt` of them.  Mostly those
// are two tensors, whose addresses are then known at once; of more, the next
// one that an element lies in is looked up among the rest unless it is the next
// of all (a run of empty tensors can be of any length: two of 20,000 inside
// slots, unpack of one copy 2,958 us walked one by one, 11.7 looked up).
template <int U, int ES, typename F, typename A>
__device__ __forceinline__ void each_element(const int64_t* offsets, int seg, int last, int64_t e, int cnt, A table,
                                             F f) {
    const int64_t end = offsets[seg + 1];
    if (e + cnt <= end) {
        const uintptr_t b = table(seg) + static_cast<uintptr_t>((e - offsets[seg]) * ES);
#pragma unroll
        for (int k = 0; k < U; ++k)
            if (k < cnt) f(k, b + k * ES);
    } else if (e + cnt <= offsets[seg + 2]) {
        const uintptr_t b0 = table(seg) + static_cast<uintptr_t>((e - offsets[seg]) * ES);
        const uintptr_t b1 = table(seg + 1) + static_cast<uintptr_t>((e - end) * ES);
#pragma unroll
        for (int k = 0; k < U; ++k)
            if (k < cnt) f(k, (e + k < end ? b0 : b1) + k * ES);
    } else {
        int sg = seg;
#pragma unroll
        for (int k = 0; k < U; ++k) {
            if (k >= cnt) continue;
            if (e + k >= offsets[sg + 1]) {
                ++sg;
                for (int h = last; e + k >= offsets[sg + 1];) {  // the last tensor that starts at or before e + k
                    const int mid = (sg + h + 1) >> 1;
                    if (offsets[mid] <= e + k) sg = mid; else h = mid - 1;
                }
            }
            f(k, table(sg) + static_cast<uintptr_t>((e + k - offsets[sg]) * ES));
        }
    }
}

}  // namespace
}  // namespace tc
