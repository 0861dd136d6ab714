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

// ---- Planes in field order, for the XOR/popcount kernels ----
// Bit i of field k (k = 8 tt + 2 c + jh of half tp) is bit 6 k + i of the 96 bits of the half's three words, so that plane i is
// what these words hold at the bit offsets i, i + 4, i + 2 modulo 6: three disjoint sets.  Joined and rotated by i, element k
// stands at bit 6 k modulo 32, an even one, whatever the plane.
__host__ __device__ __forceinline__ uint32_t rotate_right(uint32_t x, int s) { return (x >> (s & 31)) | (x << (-s & 31)); }
__host__ __device__ __forceinline__ uint32_t field_plane(uint32_t w0, uint32_t w1, uint32_t w2, int i)  // i = 0 .. 3
{
    const uint32_t b0 = 0x41041041u;  // bits 0 modulo 6
    return rotate_right((w0 & (b0 << i)) | (w1 & (b0 << (i < 2 ? i + 4 : i - 2))) | (w2 & (b0 << (i + 2))), i);
}
// plane i of half TP from the N words of a folded k step
template <int N, int TP>
__host__ __device__ __forceinline__ uint32_t folded_plane(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t w3, int i)
{
    return field_plane(unfold_word<N, 3 * TP>(w0, w1, w2, w3), unfold_word<N, 3 * TP + 1>(w0, w1, w2, w3),
                       unfold_word<N, 3 * TP + 2>(w0, w1, w2, w3), i);
}
// The other way round, nibbles to field order: n0 and n1 hold up to two bits of the elements tt = 0 and 1 (e = 2 c + jh) at
// bits 4 e, 4 e + 1; the result holds them at 6 (8 tt + e) modulo 32 and one above, i.e. two planes at its even and odd bits.
__host__ __device__ __forceinline__ uint32_t join_in_field_order(uint32_t n0, uint32_t n1)
{
    auto spread = [](uint32_t v) {  // 4 e -> 6 e modulo 32: 2 e up, by the binary digits of e
        v = (v & 0x03030303u) | ((v << 2) & 0xc0c0c0c0u);
        v = (v & 0x00c300c3u) | (rotate_right(v, 28) & 0x300c300cu);
        return (v & 0x000c30c3u) | (rotate_right(v, 24) & 0xc3000c30u);
    };
    return spread(n0) | rotate_right(spread(n1), 16);
}
// the same in the common form: element (tt, jh, c) at bits 8 c + 4 jh + 2 tt, one above
__host__ __device__ __forceinline__ uint32_t join_in_common_order(uint32_t n0, uint32_t n1) { return n0 | (n1 << 2); }
constexpr uint32_t kEvenBits = 0x55555555u;

}  // namespace apmm
