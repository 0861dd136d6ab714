// Codes out of 6-bit fields (apmm_layout.h: field form and, unfolded, the folded form), for the kernels that want bytes,
// nibbles or single planes.
#pragma once
#include <hip/hip_runtime.h>

#include "apmm_layout.h"

namespace apmm {

// The three field words w0 .. w2 of half tp of a k step hold field 8 tt + 2 c + jh at bit 48 tt + 12 c + 6 jh.  Byte c of the
// result is that field: two windows of 32 bits, 12 bits apart, hold the fields of even and odd c at their bits 0 and 24.
template <int TT, int JH>
__device__ __forceinline__ uint32_t field_dword(uint32_t w0, uint32_t w1, uint32_t w2)
{
    constexpr int at = 48 * TT + 6 * JH, next = at + 12;
    const uint32_t even = at < 32 ? __builtin_amdgcn_alignbit(w1, w0, at & 31) : __builtin_amdgcn_alignbit(w2, w1, at & 31);
    const uint32_t odd = next < 32 ? __builtin_amdgcn_alignbit(w1, w0, next & 31)
                       : next < 64 ? __builtin_amdgcn_alignbit(w2, w1, next & 31) : w2 >> (next & 31);
    return __builtin_amdgcn_perm(odd, even, 0x07030400u) & 0x0f0f0f0fu;
}

// The same from the N words of a folded k step
template <int N, int TP, int TT, int JH>
__device__ __forceinline__ uint32_t folded_dword(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t w3)
{
    return field_dword<TT, JH>(unfold_word<N, 3 * TP>(w0, w1, w2, w3), unfold_word<N, 3 * TP + 1>(w0, w1, w2, w3),
                               unfold_word<N, 3 * TP + 2>(w0, w1, w2, w3));
}
// nibbles 2 c + jh: the eight codes of t = 2 TP + TT
template <int N, int TP, int TT>
__device__ __forceinline__ uint32_t folded_nibbles(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t w3)
{
    return folded_dword<N, TP, TT, 0>(w0, w1, w2, w3) | (folded_dword<N, TP, TT, 1>(w0, w1, w2, w3) << 4);
}
// plane i of half TP in the common form of the XOR/popcount kernels: element (tt, jh, c) at bit 8 c + 4 jh + 2 tt
template <int N, int TP>
__device__ __forceinline__ uint32_t folded_plane(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t w3, int i)
{
    return ((folded_nibbles<N, TP, 0>(w0, w1, w2, w3) >> i) & 0x11111111u) |
           (((folded_nibbles<N, TP, 1>(w0, w1, w2, w3) >> i) & 0x11111111u) << 2);
}

}  // namespace apmm
