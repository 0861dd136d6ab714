// Pieces shared by the MFMA GEMM kernels: compile-time loops, the packed word -> operand expansion
// for the two operand formats, the workgroup -> tile map.
#pragma once
#include <cstdlib>
#include <type_traits>
#include <utility>

#include "apmm_epilogue.h"
#include "apmm_kernels.h"

namespace apmm {
namespace mfma {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v6i __attribute__((ext_vector_type(6)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));

// Compile-time loop: f(integral_constant<int, 0>) ... f(integral_constant<int, N-1>), always flattened,
// so that every index below is a constant (shift amounts, register numbers).
template <class F, int... Is>
__device__ __forceinline__ void static_for_impl(F &&f, std::integer_sequence<int, Is...>)
{
    (f(std::integral_constant<int, Is>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F &&f)
{
    static_for_impl(f, std::make_integer_sequence<int, N>{});
}

template <int C>
__device__ __forceinline__ uint32_t vec_word(const uint4 &u)
{
    return C == 0 ? u.x : C == 1 ? u.y : C == 2 ? u.z : u.w;
}
// word S[W], W = 0..7, of a pair group whose two slots are held as u0 = S[0..3], u1 = S[4..7]
template <int W>
__device__ __forceinline__ uint32_t pair_word(const uint4 &u0, const uint4 &u1)
{
    return W < 4 ? vec_word<W & 3>(u0) : vec_word<W & 3>(u1);
}

// ---- E2M1 (fp4) operands: v_mfma_scale_f32_*_f8f6f4, 32 codes per lane and MFMA = 4 dwords of 8 nibbles ----
// Pair group: the nibble is 00uu, whose E2M1 value is u/2 (patterns 0..3 are 0, 0.5, 1, 1.5: linear).
// Dword D = 2 tp + tt of k step KS comes from S[2 KS + tp], field tt of every nibble.
template <int KS, int D>
__device__ __forceinline__ uint32_t fp4_pair_dword(const uint4 &u0, const uint4 &u1)
{
    const uint32_t w = pair_word<2 * KS + D / 2>(u0, u1);
    return (D & 1) ? (w >> 2) & 0x33333333u : w & 0x33333333u;
}
// Single group: the bit of k step KS stands at position KS of every nibble of L[D].  Positions 0, 1, 2
// are the E2M1 values 0.5, 1, 2 (position 3 is the sign: moved to position 2); the MFMA's power-of-two
// operand scale takes the factor 2^KS (resp. 4) out again: add fp4_single_exponent(KS) to the exponent.
template <int KS, int D>
__device__ __forceinline__ uint32_t fp4_single_dword(const uint4 &u)
{
    const uint32_t l = vec_word<D>(u);
    return KS < 3 ? l & (0x11111111u << KS) : (l >> 1) & 0x44444444u;
}
constexpr int fp4_single_exponent(int ks) { return ks < 3 ? -ks : -2; }

// ---- Operands of an N-bit code from the raw vectors (slots) of a row and k block ----
// One or two bits: E2M1, four dwords (u / 2).  Weights of 3 or 4 bits: E2M3, six dwords (u / 8) from the folded form.
// With these E8M0 exponents (127 = 2^0) either operand counts 2 u, so that a product is 4 ua uw.
constexpr int operand_dwords(int n) { return n <= 2 ? 4 : 6; }
constexpr int operand_format(int n) { return n <= 2 ? 4 : 2; }  // E2M1, E2M3
constexpr int operand_exponent(int n, int ks) { return n == 1 ? 129 + fp4_single_exponent(ks) : n == 2 ? 129 : 131; }
template <int N> using OperandFrag = std::conditional_t<(N > 2), v6i, v4i>;
template <int N, int KS, int D>
__device__ __forceinline__ uint32_t operand_dword(const uint4 (&raw)[N])
{
    if constexpr (N == 1) return fp4_single_dword<KS, D>(raw[0]);
    else if constexpr (N == 2) return fp4_pair_dword<KS, D>(raw[0], raw[1]);
    else if constexpr (N == 3)
        return unfold_word<3, D>(pair_word<2 * KS>(raw[0], raw[1]), pair_word<2 * KS + 1>(raw[0], raw[1]), vec_word<KS>(raw[2]), 0u);
    else return unfold_word<4, D>(raw[KS].x, raw[KS].y, raw[KS].z, raw[KS].w);
}
__device__ __forceinline__ v8i widen(const v4i &v) { return v8i{v[0], v[1], v[2], v[3], 0, 0, 0, 0}; }
__device__ __forceinline__ v8i widen(const v6i &v) { return v8i{v[0], v[1], v[2], v[3], v[4], v[5], 0, 0}; }
// E2M3 operand of k step KS from the six slots of a field-form row: words 6 KS .. 6 KS + 5 of its 24, as they stand
// (or of local k step KS of half a k block from three)
template <int KS, int NS>
__device__ __forceinline__ v8i field_operand(const uint4 (&raw)[NS])
{
    constexpr int w = 6 * KS;
    return v8i{(int)vec_word<w & 3>(raw[w >> 2]), (int)vec_word<(w + 1) & 3>(raw[(w + 1) >> 2]),
               (int)vec_word<(w + 2) & 3>(raw[(w + 2) >> 2]), (int)vec_word<(w + 3) & 3>(raw[(w + 3) >> 2]),
               (int)vec_word<(w + 4) & 3>(raw[(w + 4) >> 2]), (int)vec_word<(w + 5) & 3>(raw[(w + 5) >> 2]), 0, 0};
}
// The same for local k step KS of half a k block.  The middle slot of the three belongs half to either k step: `mid` is this step's
// half of it, copied a step ahead (copy_here).  Left to itself the compiler makes these copies right behind the loads, each behind
// a wait, and the look-ahead is lost.
template <int KS, int NS>
__device__ __forceinline__ v8i field_operand(const uint4 (&raw)[NS], const uint2 &mid)
{
    const uint4 &own = raw[3 * (KS / 2) + 2 * (KS & 1)];
    if constexpr (KS & 1) return v8i{(int)mid.x, (int)mid.y, (int)own.x, (int)own.y, (int)own.z, (int)own.w, 0, 0};
    else return v8i{(int)own.x, (int)own.y, (int)own.z, (int)own.w, (int)mid.x, (int)mid.y, 0, 0};
}

// ---- The same for stages of half a k block: k steps 2 H, 2 H + 1 (KSL = 0, 1), whose words are these slots ----
constexpr int half_slots(int n, bool field) { return field ? 3 : n <= 2 ? 1 : 2; }
constexpr int half_slot(int n, bool field, int h, int i) { return field ? 3 * h + i : n == 1 ? 0 : n == 2 ? h : n == 3 ? (i == 0 ? h : 2) : 2 * h + i; }
template <int N, int H, int KSL, int D, int NS>
__device__ __forceinline__ uint32_t half_operand_dword(const uint4 (&raw)[NS])
{
    if constexpr (N == 1) return fp4_single_dword<2 * H + KSL, D>(raw[0]);
    else if constexpr (N == 2) return (D & 1) ? (vec_word<2 * KSL + D / 2>(raw[0]) >> 2) & 0x33333333u : vec_word<2 * KSL + D / 2>(raw[0]) & 0x33333333u;
    else if constexpr (N == 3)
        return unfold_word<3, D>(vec_word<2 * KSL>(raw[0]), vec_word<2 * KSL + 1>(raw[0]), vec_word<2 * H + KSL>(raw[NS - 1]), 0u);
    else return unfold_word<4, D>(raw[KSL].x, raw[KSL].y, raw[KSL].z, raw[KSL].w);
}

// x / d for the tile maps, where the way to the first request counts: the launcher passes ceil(2^32 / d), or 0 where d = 1 or x d does not
// stay below 2^32 (then the quotient of x and this could be one too high).  A division takes 25 instructions in a row.
inline uint32_t divisor_magic(int64_t d, int64_t most_x)
{
    return d > 1 && d * most_x < ((int64_t)1 << 32) ? (uint32_t)((((int64_t)1 << 32) + d - 1) / d) : 0u;
}
__device__ __forceinline__ uint32_t quotient(uint32_t x, uint32_t d, uint32_t magic)
{
    if (magic != 0) return __umulhi(x, magic);
    return d <= 1 ? x : x / d;
}
// k blocks of a row
__device__ __forceinline__ uint32_t padded_k_blocks(uint32_t k) { return (k + (kKPad - 1)) / kKPad * (kKPad / kKBlock); }

// Workgroups are dealt round-robin to the 8 XCDs; give each XCD a contiguous run of tiles so that
// the packed rows it re-reads stay in its own L2.
__device__ __forceinline__ int xcd_tile_id(int block, int tiles_total)
{
    if ((tiles_total & 7) == 0) return (block & 7) * (tiles_total >> 3) + (block >> 3);
    return block;
}

// ---- Streaming stores of inner tiles: the launcher's choice, the kernels' last argument ----
// A streaming store leaves the operands in L2 alone and is written back early, but a line that it fills only in part is written in
// parts: rows that do not begin at a line (N no multiple of 32, or an output that begins elsewhere) share their lines with the wave
// tile next to them.  Plain stores meet in L2.  Both outputs, all streaming against all plain, operands and outputs in rotation:
// 1500 x 11010 x 512 W2A2 57 against 30 us, 2048 x 4098 x 512 26 / 16, 1536 x 5002 x 512 24 / 18; W8A8 1500 x 5002 x 512 1.7 times.
// The outputs of a call that fit the L2 of all XCDs (32 MB) well, but are not small, are the exception: 3 - 10 % faster streaming at 8 to
// 22 MB (an int32 output of half lines up to 30), as much slower below (203 x 4098 x 512 both 6 %).
struct OutputRows {
    int64_t bytes;  // of all outputs of the call
    bool both, whole, half_lines;  // whole: every row begins and ends at a line (fp16: at half of one, the run of a wave's row); half_lines: int32 alone
    explicit OutputRows(const GemmArgs &g)
        : bytes(g.M * g.N * ((g.c_i32 ? 4 : 0) + (g.c_f16 ? 2 : 0))), both(g.c_i32 && g.c_f16),
          whole((g.N & 31) == 0 && (reinterpret_cast<uintptr_t>(g.c_i32) & 127) == 0 && (reinterpret_cast<uintptr_t>(g.c_f16) & 63) == 0),
          half_lines((g.N & 15) == 0 && !g.c_f16)
    {
    }
    bool up_to_l2(int64_t most) const { return bytes < (half_lines ? 30000000 : most); }
    bool fit_l2(int64_t most = 22000000) const { return bytes >= 8000000 && up_to_l2(most); }
};

}  // namespace mfma
}  // namespace apmm
