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
// A unit is the 64 codes of k steps 2 kk, 2 kk + 1 of one row and k block: up to four 16-byte loads, and four 16-byte
// operand chunks ks, tp whose word 2 tt + jh, byte c is element (ks, 2 tp + tt, jh, c): the order of the elements.
#pragma once
#include <hip/hip_runtime.h>

#include "apmm_layout.h"

namespace apmm {
namespace i8 {

constexpr int kSlotVec = kPlaneWords / 4;  // uint4 between slots of a tile

struct Form {
    int n;       // bits
    bool field;  // 6-bit fields (activations of 3 and 4 bits)
    __host__ __device__ int slots() const { return field ? 6 : n; }
};

__host__ __device__ inline uint32_t code_bias(int n) { return n == 8 ? 128u : 0u; }                       // z
__host__ __device__ inline uint32_t value_offset(int n) { return n == 8 ? ~0u : (1u << n) - 1u; }         // c' modulo 2^32

// Loads of unit kk (slot 0 of the row and k block at `s`).  Forms of fewer than four loads repeat one, so that the
// number of requests in flight does not depend on the form: the wait for a set of loads may then leave exactly the
// sets requested after it outstanding.
__device__ __forceinline__ void load_unit(Form f, int kk, const uint4 *__restrict__ s, uint4 (&raw)[4])
{
    int o0, o1, o2, o3;
    if (f.field) {
        o0 = 3 * kk; o1 = o0 + 1; o2 = o0 + 2; o3 = o2;
    } else if (byte_form(f.n)) {
        o0 = 4 * kk; o1 = o0 + 1; o2 = o0 + 2; o3 = o0 + 3;
    } else if (nibble_form(f.n)) {
        o0 = 2 * kk; o1 = o0 + 1; o2 = f.n >= 6 ? 4 + kk : o1; o3 = has_single_group(f.n) ? f.n - 1 : o2;
    } else {
        o0 = f.n == 1 ? 0 : kk; o1 = f.n == 4 ? 2 + kk : o0; o2 = o1; o3 = has_single_group(f.n) ? f.n - 1 : o2;
    }
    raw[0] = s[o0 * kSlotVec];
    raw[1] = s[o1 * kSlotVec];
    raw[2] = s[o2 * kSlotVec];
    raw[3] = s[o3 * kSlotVec];
}

__device__ __forceinline__ uint32_t word_of(const uint4 &v, int i) { return i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w; }

// pair group in S[4 kk ..] (`s`): dword (e, tp, tt, jh) has its two bits at the bottom of every byte
__device__ __forceinline__ uint32_t pair_bytes(const uint4 &s, int e, int tp, int tt, int jh)
{
    return (word_of(s, 2 * e + tp) >> (4 * jh + 2 * tt)) & 0x03030303u;
}
// single group (`l`), ks = 2 kk + e
__device__ __forceinline__ uint32_t single_bytes(const uint4 &l, int ks, int tp, int tt, int jh)
{
    return (word_of(l, 2 * tp + tt) >> (4 * jh + ks)) & 0x01010101u;
}

// chunk[2 e + tp] = operand chunk of k step 2 kk + e, half tp.  The form is uniform over the wave.
__device__ __forceinline__ void expand_unit(Form f, int kk, const uint4 (&raw)[4], uint4 (&chunk)[4])
{
    auto fill = [&](auto dword) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int tp = 0; tp < 2; ++tp)
                chunk[2 * e + tp] = make_uint4(dword(e, tp, 0, 0), dword(e, tp, 0, 1), dword(e, tp, 1, 0), dword(e, tp, 1, 1));
    };
    if (f.field) {
        const uint32_t w[12] = {raw[0].x, raw[0].y, raw[0].z, raw[0].w, raw[1].x, raw[1].y,
                                raw[1].z, raw[1].w, raw[2].x, raw[2].y, raw[2].z, raw[2].w};
        // 48 bits of (e, t): byte c of dword jh is the field at bit 12 c + 6 jh
        fill([&](int e, int tp, int tt, int jh) __attribute__((always_inline)) {
            const uint32_t *d = w + 6 * e + 3 * tp;
            const uint64_t bits = (tt == 0 ? (uint64_t)d[0] | ((uint64_t)(d[1] & 0xffffu) << 32)
                                           : (uint64_t)(d[1] >> 16) | ((uint64_t)d[2] << 16)) >> (6 * jh);
            const uint32_t lo = (uint32_t)bits;
            return (lo & 0x3fu) | ((lo >> 4) & 0x3f00u) | ((lo >> 8) & 0x3f0000u) | ((uint32_t)(bits >> 12) & 0x3f000000u);
        });
        return;
    }
    switch (f.n) {
    case 1:
        fill([&](int e, int tp, int tt, int jh) __attribute__((always_inline)) { return single_bytes(raw[3], 2 * kk + e, tp, tt, jh); });
        break;
    case 2:
        fill([&](int e, int tp, int tt, int jh) __attribute__((always_inline)) { return pair_bytes(raw[0], e, tp, tt, jh); });
        break;
    case 3:
        fill([&](int e, int tp, int tt, int jh) __attribute__((always_inline)) {
            return pair_bytes(raw[0], e, tp, tt, jh) | (single_bytes(raw[3], 2 * kk + e, tp, tt, jh) << 2);
        });
        break;
    case 4:
        fill([&](int e, int tp, int tt, int jh) __attribute__((always_inline)) {
            return pair_bytes(raw[0], e, tp, tt, jh) | (pair_bytes(raw[1], e, tp, tt, jh) << 2);
        });
        break;
    case 8:
#pragma unroll
        for (int i = 0; i < 4; ++i) chunk[i] = raw[i];
        break;
    default:  // 5, 6, 7: nibble words N[4 ks + t] in raw[e], then the pair group of bits 4, 5 and / or the single top bit
        fill([&](int e, int tp, int tt, int jh) __attribute__((always_inline)) {
            return (word_of(raw[e], 2 * tp + tt) >> (4 * jh)) & 0x0f0f0f0fu;
        });
        auto add = [&](auto dword) __attribute__((always_inline)) {
#pragma unroll
            for (int e = 0; e < 2; ++e)
#pragma unroll
                for (int tp = 0; tp < 2; ++tp) {
                    uint4 &c = chunk[2 * e + tp];
                    c = make_uint4(c.x | dword(e, tp, 0, 0), c.y | dword(e, tp, 0, 1), c.z | dword(e, tp, 1, 0), c.w | dword(e, tp, 1, 1));
                }
        };
        if (f.n >= 6) add([&](int e, int tp, int tt, int jh) __attribute__((always_inline)) { return pair_bytes(raw[2], e, tp, tt, jh) << 4; });
        if (f.n == 5) add([&](int e, int tp, int tt, int jh) __attribute__((always_inline)) { return single_bytes(raw[3], 2 * kk + e, tp, tt, jh) << 4; });
        if (f.n == 7) add([&](int e, int tp, int tt, int jh) __attribute__((always_inline)) { return single_bytes(raw[3], 2 * kk + e, tp, tt, jh) << 6; });
        break;
    }
}

}  // namespace i8
}  // namespace apmm
