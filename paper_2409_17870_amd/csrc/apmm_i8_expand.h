// Packed words -> int8 matrix-unit operands, for every packed form (apmm_layout.h).
//
// The codes themselves are the operands: u for up to 7 bits, u - 128 for 8 bits (which do not fit a signed byte
// otherwise).  With u = u' + z (z = 128 for 8 bits, else 0) the value of an n-bit code is 2u - (2^n - 1) = 2u' - c',
// c' = 2^n - 1 - 2z, i.e. -1 for 8 bits, and the recovery of C from S = sum ua' uw' is that of the other matrix-unit
// kernels with c' and the sums of u' in the place of 2^n - 1 and the code sums:
//   C = 4 S - 2 cw' PA' - 2 ca' PW' + K' ca' cw' - (K' - K)(2^p - 1)(2^q - 1),      K' = K padded,
// where the last term takes the padding out again (its codes are all ones, values 2^n - 1).  Everything is computed
// modulo 2^32; the true C fits 32 bits (checked on the host).
//
// The bytes of an operand chunk are elements in their own order: word 2 tt + jh, byte c of chunk (ks, tp) is element
// (ks, 2 tp + tt, jh, c), 16 consecutive codes.
#pragma once
#include <hip/hip_runtime.h>

#include "apmm_fields.h"

namespace apmm {
namespace i8 {

__host__ __device__ inline uint32_t code_bias(int n) { return n == 8 ? 128u : 0u; }                       // z
__host__ __device__ inline uint32_t value_offset(int n) { return n == 8 ? ~0u : (1u << n) - 1u; }         // c' modulo 2^32

// Compile-time forms.  1, 2: that many bits in the group form; 3, 4: weights in the folded form.
constexpr int kNibbles = 5, kFields = 6, kBytes = 8;  // 5 .. 7 bits; 6-bit fields (activations of 3, 4 bits); 8 bits
constexpr int form_loads(int form) { return form <= 2 ? 1 : form <= 4 ? 2 : form == kFields ? 3 : 4; }

// Run-time part of an operand: slots per row and k block; for kNibbles where the bits above the nibble are.
struct Operand {
    int slots;
    int pair_slot, single_slot;          // kNibbles: slots of S of bits 4, 5 (first of two) and of the single top bit
    uint32_t pair_mask, single_mask;     // 0 where the width has no such group
    int single_pos;                      // bit position of the single group
};
template <int FORM>
__device__ __forceinline__ Operand make_operand(int n)
{
    Operand o = {FORM == kFields ? 6 : FORM == kNibbles ? n : FORM, 0, 0, 0, 0, 0};
    if constexpr (FORM == kNibbles) {
        if (n >= 6) { o.pair_slot = 4; o.pair_mask = 0x30303030u; }
        if (n & 1) { o.single_slot = n - 1; o.single_mask = 0x01010101u; o.single_pos = n - 1; }
    }
    return o;
}

// shift right by S, or left for a negative S
template <int S>
__device__ __forceinline__ uint32_t shifted(uint32_t x)
{
    return S >= 0 ? x >> (S >= 0 ? S : 0) : x << (S < 0 ? -S : 0);
}

}  // namespace i8
}  // namespace apmm
