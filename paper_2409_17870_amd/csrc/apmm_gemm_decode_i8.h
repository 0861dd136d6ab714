// Small-M kernel on the int8 matrix operations: up to 64 tokens, a code of more than four bits on either side (and
// packed 3- and 4-bit codes at a K beyond the exactness bound of the fp4 kernels).
//
// Algebra: apmm_i8_expand.h.  Split of the work as in the fp4 small-M kernel: a workgroup owns 16 RT output channels and
// all tokens, its eight waves split K, partial sums meet in LDS, nothing is staged and no barrier stands before the k
// loop.  A wave takes one k block per step, lane (r16, ks) the 32 codes of row (or token) r16 in k step ks:
//   v_mfma_i32_16x16x64_i8: A = 16 weight rows x 64 k, B = 64 k x 16 tokens; MFMA tp of a block multiplies the chunks
//   (ks, tp) of all four k steps.  An operand chunk is 16 consecutive codes, so unpacked activation codes are the operand
//   as they stand (one XOR for 8 bits, one AND for fewer): no exchange between lanes, and the four lanes of a token read
//   one 128-byte line.  Their sums PA' come from one more MFMA against a fragment of ones.
// U blocks per step are requested one step ahead.
//
// What bounds it: the launch and the round trip of its loads, then the weights' bytes and (from codes) the tokens' lines,
// which every workgroup reads for itself.  The XOR/popcount kernel that served up to 16 tokens of 5 .. 8 bits is bound by
// the vector ALU, p q plane pairs for every token; 17 .. 64 tokens and wide weights took 64 x 128 tiles on a few CUs.
// Measured (fp16 output, one launch inside a graph, weights in rotation over 400 MB; M x N x K): W4A8 from codes 8 x 11008 x
// 4096 63.5 -> 8.4 us, 16 x 4096 x 4096 5.4 us; W8A8 packed 8 x 4096 x 4096 5.4 us (3.1 TB/s), 32 x 4096 x 4096 18.0 -> 6.4 us,
// 64 x 4096 x 11008 42.4 -> 17.8 us.
#pragma once
#include <hip/hip_ext.h>

#include "apmm_decode_common.h"
#include "apmm_i8_expand.h"

namespace apmm {
namespace i8 {

using mfma::static_for;
using mfma::vec_word;
using mfma::v4i;

constexpr int kCodes = 9;  // unpacked codes, one per byte

// What a lane loads of its 32 codes: whole slot vectors, two-word halves of them, single words.
template <int FORM>
struct LaneUnit {
    static constexpr int kVecs = FORM == 1 || FORM == 4 ? 1 : FORM == kNibbles || FORM == kBytes || FORM == kCodes ? 2 : 0;
    static constexpr int kHalves = FORM == 2 || FORM == 3 || FORM == kNibbles ? 1 : FORM == kFields ? 3 : 0;
    static constexpr int kSingles = FORM == 3 ? 1 : 0;
    static constexpr int kWords = 4 * kVecs + 2 * kHalves + kSingles;
    uint32_t s[kSingles ? kSingles : 1];
    uint4 v[kVecs ? kVecs : 1];
    uint2 h[kHalves ? kHalves : 1];
};

// k blocks per step, whose words are held twice: two where that leaves two workgroups on a CU (128 registers).  (Four for one
// tile of narrow forms, the earlier rule, spilled registers in three of them and loaded up to 64 blocks where K has 40: one
// token from codes 5120 x 5120 W4A5 7.3 -> 6.3 us, 5120 x 13824 13.9 -> 12.4 us; packed W1A8 1000 x 2048 2.9 -> 2.5 us; the
// median over sizes from 1000 x 2048 to 13824 x 5120 is 5 - 15 % less, the worst W2A8 8192 x 8192, 5.9 -> 6.2 us.)
constexpr int unit_steps(int words) { return words <= 20 ? 2 : 1; }

// `src`: the k block (a scalar), `row`: bytes from there to word 0 of slot 0 of the lane's row
template <int FORM>
__device__ __forceinline__ void load_unit(const Operand &o, const char *src, uint32_t row, uint32_t ks, LaneUnit<FORM> &u)
{
    constexpr uint32_t kSlotBytes = kPlaneWords * 4;
    auto vec = [&](uint32_t slot) __attribute__((always_inline)) { return *reinterpret_cast<const uint4 *>(src + (row + slot * kSlotBytes)); };
    auto words = [&](uint32_t w) __attribute__((always_inline)) {  // words w, w + 1 (w even) of the row, four to a slot
        return *reinterpret_cast<const uint2 *>(src + (row + (w >> 2) * kSlotBytes + (w & 3) * 4));
    };
    if constexpr (FORM == 1) {
        u.v[0] = vec(0);
    } else if constexpr (FORM == 2) {
        u.h[0] = words(2 * ks);
    } else if constexpr (FORM == 3) {
        u.h[0] = words(2 * ks);
        u.s[0] = *reinterpret_cast<const uint32_t *>(src + (row + 2 * kSlotBytes + ks * 4));
    } else if constexpr (FORM == 4) {
        u.v[0] = vec(ks);
    } else if constexpr (FORM == kNibbles) {
        u.v[0] = vec(ks);
        u.h[0] = words(4 * o.pair_slot + 2 * ks);
        u.v[1] = vec(o.single_slot);
    } else if constexpr (FORM == kFields) {
#pragma unroll
        for (int i = 0; i < 3; ++i) u.h[i] = words(6 * ks + 2 * i);
    } else {
        u.v[0] = vec(2 * ks);
        u.v[1] = vec(2 * ks + 1);
    }
}

template <int W>
__device__ __forceinline__ uint32_t half_word(const uint2 &u) { return W ? u.y : u.x; }

// dword D = 2 tt + jh of chunk tp of the lane's 32 codes
template <int FORM, int TP, int D>
__device__ __forceinline__ uint32_t unit_dword(const Operand &o, const LaneUnit<FORM> &u, int ks)
{
    constexpr int tt = D / 2, jh = D % 2, t = 2 * TP + tt, pair_at = 4 * jh + 2 * tt;
    if constexpr (FORM == 1) {
        return ((vec_word<t>(u.v[0]) >> ks) >> (4 * jh)) & 0x01010101u;
    } else if constexpr (FORM == 2) {
        return (half_word<TP>(u.h[0]) >> pair_at) & 0x03030303u;
    } else if constexpr (FORM == 3) {
        return folded_dword<3, TP, tt, jh>(u.h[0].x, u.h[0].y, u.s[0], 0u);
    } else if constexpr (FORM == 4) {
        return folded_dword<4, TP, tt, jh>(u.v[0].x, u.v[0].y, u.v[0].z, u.v[0].w);
    } else if constexpr (FORM == kNibbles) {
        uint32_t v = (vec_word<t>(u.v[0]) >> (4 * jh)) & 0x0f0f0f0fu;
        v |= shifted<pair_at - 4>(half_word<TP>(u.h[0])) & o.pair_mask;
        return v | ((((vec_word<t>(u.v[1]) >> ks) >> (4 * jh)) & o.single_mask) << o.single_pos);
    } else if constexpr (FORM == kFields) {
        return field_dword<tt, jh>(half_word<(3 * TP) % 2>(u.h[(3 * TP) / 2]), half_word<(3 * TP + 1) % 2>(u.h[(3 * TP + 1) / 2]),
                                   half_word<(3 * TP + 2) % 2>(u.h[(3 * TP + 2) / 2]));
    } else {
        return vec_word<D>(u.v[TP]);
    }
}

template <int FA, int FB, int TT, int RT>
__global__ __launch_bounds__(kDecodeThreads, TT * RT == 1 ? 4 : 2)  // waves per SIMD aimed at
void gemm_decode_i8_kernel(const uint32_t *w_arg, const void *a_arg, int n_arg, int k_arg, uint32_t misc_arg /* M | problems << 12 */,
                           int pq_arg /* p | q << 8 */, uint16_t *cf_arg, int32_t *ci_arg, const uint16_t *ws_arg,
                           const uint16_t *as_arg, GroupArgs ga)
{
    constexpr bool CODES = FA == kCodes;
    constexpr int W = kDecodeWaves, U = unit_steps(RT * LaneUnit<FB>::kWords + TT * LaneUnit<FA>::kWords);
    constexpr int OUTS = (TT * RT * 256 + kDecodeThreads - 1) / kDecodeThreads;
    extern __shared__ __align__(16) uint8_t lds_raw[];
    DecodeProblem pr = {w_arg, a_arg, n_arg, k_arg, (int64_t)(misc_arg & 0xfffu), cf_arg, ci_arg, ws_arg, as_arg};
    const int block = pick_problem(pr, misc_arg, ga);
    const int p = pq_arg & 0xff, q = pq_arg >> 8;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15, ks = lane >> 4;
    // (the way to the first request as in the fp4 small-M kernel: bases are scalars, a lane's part of an address is 32 bits; the channels
    // of a workgroup and the tokens of two tiles lie in one row block, whose rows past the operand's are zero words.  W4A8 from codes 8 x 11008 x
    // 4096 9.3 -> 9.1 us, W8A8 packed 8 x 4096 x 4096 5.4 -> 5.2, W8A7 40 x 1000 x 2000 6.1 -> 5.7)
    const int n0 = block * (kRowsPerWg * RT), M = (int)pr.M, N = (int)pr.N;
    const int nkb = (int)mfma::padded_k_blocks((uint32_t)pr.K);
    const Operand ob = make_operand<FB>(q), oa = make_operand<CODES ? 1 : FA>(p);

    constexpr uint32_t kSlotBytes = kPlaneWords * 4;
    const uint32_t w_row = ((uint32_t)(n0 & 16) + r16) * 16, a_row = r16 * 16;
    const char *w_base = reinterpret_cast<const char *>(pr.w) + (uint64_t)(((uint32_t)n0 >> 5) * (uint32_t)nkb) * (ob.slots * kSlotBytes);
    const uint8_t *crow[TT];
#pragma unroll
    for (int tt = 0; tt < TT; ++tt)
        if constexpr (CODES) crow[tt] = static_cast<const uint8_t *>(pr.a) + (int64_t)min(tt * 16 + r16, M - 1) * pr.K;  // tokens past M: the last one, never stored
    const int last = (int)pr.K - 16;  // CODES: K >= 16 (the launcher's rule)

    LaneUnit<FB> wn[U][RT];
    LaneUnit<FA> an[U][TT];
    // Four token tiles of several loads each: the block's place as an opaque scalar per tile, or the compiler asks for the tiles in pairs and carries
    // six 64-bit lane addresses through the k loop instead of three (33 - 64 tokens, W8A5 64 x 1024 x 16384 26.7 -> 24.3 us, 64 x 4096 x 11008 21.1 ->
    // 19.8, W4A5 27.0 -> 24.6, W1A5 24.7 -> 23.2, W5A3 0.86 - 0.97 of the time).  Nibbles on both sides: 1.00 - 1.06, left alone.
    constexpr bool SCALAR_BLOCK = TT == 4 && (FA == kFields || (FA == kNibbles && FB != kNibbles));
    auto load_block = [&](int u, int kb) __attribute__((always_inline)) {
        kb = kb < nkb ? kb : nkb - 1;  // (blocks past the end are loaded from the last one and not multiplied)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) load_unit<FB>(ob, w_base + (uint64_t)kb * (ob.slots * kSlotBytes), w_row + rt * 256, ks, wn[u][rt]);
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) {
            if constexpr (CODES) {
#pragma unroll
                for (int tp = 0; tp < 2; ++tp) {
                    const int k0 = kb * kKBlock + 32 * ks + 16 * tp;
                    const Codes16 c = *reinterpret_cast<const Codes16 *>(crow[tt] + (k0 < last ? k0 : last));
                    an[u][tt].v[tp] = make_uint4(c.x, c.y, c.z, c.w);
                }
            } else {
                uint64_t block_at = (uint64_t)((tt / 2) * nkb + kb) * (oa.slots * kSlotBytes);
                if constexpr (SCALAR_BLOCK) asm volatile("" : "+s"(block_at));
                load_unit<FA>(oa, static_cast<const char *>(pr.a) + block_at, a_row + (tt & 1) * 256, ks, an[u][tt]);
            }
        }
    };
#pragma unroll
    for (int u = 0; u < U; ++u) load_block(u, wave + u * W);

    // what only the final store needs is requested behind the first operands and kept as loaded
    bool out_ok[OUTS];
    int out_m[OUTS], out_n[OUTS];
    uint32_t out_sa_bits[OUTS], out_sw_bits[OUTS], out_pa[OUTS], out_pw[OUTS];
    {
        const uint32_t rows_a = (M + 31u) & ~31u, rows_b = (N + 31u) & ~31u;
        const int32_t *w_sum = reinterpret_cast<const int32_t *>(pr.w) + (uint64_t)rows_b * nkb * (ob.slots * 4);
        const int32_t *a_sum = CODES ? w_sum : static_cast<const int32_t *>(pr.a) + (uint64_t)rows_a * nkb * (oa.slots * 4);
        const uint16_t *sa = pr.a_scale ? pr.a_scale : reinterpret_cast<const uint16_t *>(pr.w), *sw = pr.w_scale ? pr.w_scale : reinterpret_cast<const uint16_t *>(pr.w);
        const uint32_t last_m = pr.a_scale ? M - 1 : 0, last_n = pr.w_scale ? N - 1 : 0;
#pragma unroll
        for (int o = 0; o < OUTS; ++o) {
            // element (tile t = e / 256, register v, lane l) of the accumulators: row 4 (l / 16) + v (channel), column l % 16 (token)
            // (a wave without a tile, where there are fewer than two, stands at the last one and stores nothing)
            const int t_all = (wave >> 2) + o * (W / 4), t = t_all < TT * RT ? t_all : TT * RT - 1;
            out_m[o] = (t % TT) * 16 + r16;
            out_n[o] = n0 + (t / TT) * 16 + (wave & 3) + 4 * ks;
            out_ok[o] = t_all < TT * RT && out_m[o] < M && out_n[o] < N;
            out_pa[o] = CODES ? 0u : (uint32_t)a_sum[(uint32_t)out_m[o]];
            out_pw[o] = (uint32_t)w_sum[(uint32_t)out_n[o]];
            out_sa_bits[o] = sa[min((uint32_t)out_m[o], last_m)];
            out_sw_bits[o] = sw[min((uint32_t)out_n[o], last_n)];
        }
    }

    v4i acc[RT][TT], acc_pa[TT];
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) {
        acc_pa[tt] = v4i{0, 0, 0, 0};
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) acc[rt][tt] = v4i{0, 0, 0, 0};
    }
    const uint32_t code_mask = p == 8 ? ~0u : 0x01010101u * ((1u << p) - 1u), flip = p == 8 ? 0x80808080u : 0u;
    const bool ragged = (pr.K & 15) != 0;

    for (int kb0 = wave; kb0 < nkb; kb0 += U * W) {
        LaneUnit<FB> wc[U][RT];
        LaneUnit<FA> ac[U][TT];
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) wc[u][rt] = wn[u][rt];
#pragma unroll
            for (int tt = 0; tt < TT; ++tt) ac[u][tt] = an[u][tt];
        }
        if (kb0 + U * W < nkb) {
#pragma unroll
            for (int u = 0; u < U; ++u) load_block(u, kb0 + (U + u) * W);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int kb = kb0 + u * W;
            if (kb >= nkb) continue;  // uniform over the wave
            if constexpr (CODES) {
#pragma unroll
                for (int tt = 0; tt < TT; ++tt)
#pragma unroll
                    for (int tp = 0; tp < 2; ++tp) {
                        const int past = kb * kKBlock + 32 * ks + 16 * tp - last;
                        uint4 c = ac[u][tt].v[tp];
                        if (ragged) c = shift_past(c, past);
                        else if (past > 0) c = make_uint4(~0u, ~0u, ~0u, ~0u);
                        ac[u][tt].v[tp] = make_uint4((c.x & code_mask) ^ flip, (c.y & code_mask) ^ flip, (c.z & code_mask) ^ flip,
                                                     (c.w & code_mask) ^ flip);
                    }
            }
            static_for<2>([&](auto tp_c) __attribute__((always_inline)) {
                constexpr int tp = decltype(tp_c)::value;
                v4i a[TT], w[RT];
                static_for<4>([&](auto d_c) __attribute__((always_inline)) {
                    constexpr int d = decltype(d_c)::value;
#pragma unroll
                    for (int tt = 0; tt < TT; ++tt) a[tt][d] = (int)unit_dword<FA, tp, d>(oa, ac[u][tt], ks);
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt) w[rt][d] = (int)unit_dword<FB, tp, d>(ob, wc[u][rt], ks);
                });
#pragma unroll
                for (int tt = 0; tt < TT; ++tt) {
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt) acc[rt][tt] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w[rt], a[tt], acc[rt][tt], 0, 0, 0);
                    if constexpr (CODES)
                        acc_pa[tt] = __builtin_amdgcn_mfma_i32_16x16x64_i8(v4i{0x01010101, 0x01010101, 0x01010101, 0x01010101}, a[tt],
                                                                           acc_pa[tt], 0, 0, 0);
                }
            });
        }
    }

    // reduce over the waves through LDS: part[wave][tile t][v][lane], and (CODES) the sums pa[wave][token]
    uint32_t *part = reinterpret_cast<uint32_t *>(lds_raw), *pa_lds = part + W * RT * TT * 256;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int tt = 0; tt < TT; ++tt)
#pragma unroll
            for (int v = 0; v < 4; ++v) part[((wave * RT * TT + rt * TT + tt) * 4 + v) * 64 + lane] = (uint32_t)acc[rt][tt][v];
    if constexpr (CODES) {
#pragma unroll
        for (int tt = 0; tt < TT; ++tt)
            if (lane < 16) pa_lds[(wave * TT + tt) * 16 + lane] = (uint32_t)acc_pa[tt][0];  // row 0, token = lane
    }
    __syncthreads();
    const uint32_t ca = value_offset(p), cw = value_offset(q), k_pad = (uint32_t)nkb * kKBlock;
    const uint32_t full = k_pad * ca * cw - (k_pad - (uint32_t)pr.K) * ((1u << p) - 1u) * ((1u << q) - 1u);
#pragma unroll
    for (int o = 0; o < OUTS; ++o) {
        if (!out_ok[o]) continue;
        const int e = tid + o * kDecodeThreads;  // = (t * 4 + v) * 64 + l
        uint32_t s = 0, pa = 0;
#pragma unroll
        for (int w8 = 0; w8 < W; ++w8) {
            s += part[w8 * RT * TT * 256 + e];
            if constexpr (CODES) pa += pa_lds[w8 * TT * 16 + out_m[o]];
        }
        if constexpr (!CODES) pa = use_here(out_pa[o]) - code_bias(p) * k_pad;
        const uint32_t pw = use_here(out_pw[o]) - code_bias(q) * k_pad;
        const int32_t c = (int32_t)(4u * s - 2u * cw * pa - 2u * ca * pw + full);
        const uint32_t sa_bits = pr.a_scale ? use_here(out_sa_bits[o]) : 0x3c00u;  // 1.0
        const uint32_t sw_bits = pr.w_scale ? use_here(out_sw_bits[o]) : 0x3c00u;
        const int64_t at = (int64_t)out_m[o] * N + out_n[o];
        if (pr.c_i32) pr.c_i32[at] = c;
        if (pr.c_f16)
            pr.c_f16[at] = float_to_half_bits((float)c * half_bits_to_float((uint16_t)sa_bits) * half_bits_to_float((uint16_t)sw_bits));
    }
}

template <int FA, int FB, int TT, int RT>
hipError_t launch_decode_variant(const GroupArgs &ga, hipStream_t stream)
{
    const GemmArgs &g = ga.g[0];
    const size_t lds = (size_t)kDecodeWaves * TT * (RT * 256 + 16) * 4;
    const dim3 grid((unsigned)ga.wg_end[ga.count - 1]), block(kDecodeThreads);
    const void *a = FA == kCodes ? static_cast<const void *>(g.a_codes) : static_cast<const void *>(g.a);
    const uint32_t misc = (uint32_t)g.M | ((uint32_t)ga.count << 12);
    const int pq = g.p | (g.q << 8);
    const auto kernel = gemm_decode_i8_kernel<FA, FB, TT, RT>;
    note_kernel("gemm_decode_i8_kernel<%d,%d,%d,%d,%s>", g.p, g.q, TT, RT, FA == kCodes ? "codes" : "packed");
    const KernelTiming timing = take_kernel_timing();
    if (timing.start || timing.stop)
        hipExtLaunchKernelGGL(kernel, grid, block, lds, stream, timing.start, timing.stop, 0, g.w, a, (int)g.N, (int)g.K, misc, pq,
                              g.c_f16, g.c_i32, g.w_scale, g.a_scale, ga);
    else
        hipLaunchKernelGGL(kernel, grid, block, lds, stream, g.w, a, (int)g.N, (int)g.K, misc, pq, g.c_f16, g.c_i32, g.w_scale,
                           g.a_scale, ga);
    return hipGetLastError();
}

template <int FA, int FB>
hipError_t launch_decode_forms(const GroupArgs &ga, int tt, int rt, hipStream_t stream)
{
    if (tt == 1) return rt == 1 ? launch_decode_variant<FA, FB, 1, 1>(ga, stream) : launch_decode_variant<FA, FB, 1, 2>(ga, stream);
    if (tt == 2) return rt == 1 ? launch_decode_variant<FA, FB, 2, 1>(ga, stream) : launch_decode_variant<FA, FB, 2, 2>(ga, stream);
    return launch_decode_variant<FA, FB, 4, 1>(ga, stream);
}

// weights of any width
template <int FA>
hipError_t launch_decode_q(const GroupArgs &ga, int tt, int rt, hipStream_t stream)
{
    switch (ga.g[0].q) {
    case 1: return launch_decode_forms<FA, 1>(ga, tt, rt, stream);
    case 2: return launch_decode_forms<FA, 2>(ga, tt, rt, stream);
    case 3: return launch_decode_forms<FA, 3>(ga, tt, rt, stream);
    case 4: return launch_decode_forms<FA, 4>(ga, tt, rt, stream);
    case 8: return launch_decode_forms<FA, kBytes>(ga, tt, rt, stream);
    default: return launch_decode_forms<FA, kNibbles>(ga, tt, rt, stream);
    }
}

}  // namespace i8
}  // namespace apmm
