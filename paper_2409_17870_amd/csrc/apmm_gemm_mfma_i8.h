// Matrix-unit GEMM for codes of more than four bits (and for 3- and 4-bit codes at a K beyond the exactness bound of the
// fp4 kernels): packed words -> int8 operands in registers, v_mfma_i32_32x32x32_i8.
//
// Algebra and operand forms: apmm_i8_expand.h.  Paper Sec. 3.2's shift-and-add over plane pairs happens in front of the
// multiplier, once per operand byte; p q 1-bit products become one, accumulated exactly in int32.
//
// Every wave owns a 64 x 128 tile (2 x 4 blocks of 32 x 32).  KSPLIT: the four waves of a workgroup hold the same tile
// and a quarter of K each, and meet in LDS at the end (outputs of few tiles: 512 x 4096 is 256 of them); else 2 x 2
// waves, a 128 x 256 tile.  A stage is the 64 codes of one half kk of two k blocks (lanes 0 .. 31 hold the first,
// lanes 32 .. 63 the second): up to four 16-byte loads per row block, four MFMA k steps.  Raw words are double buffered
// in registers one stage ahead, the operand bytes of k step i + 1 are formed between the MFMAs of step i.  No LDS and
// no barrier in the k loop.
//
// What bounds it: L1.  A k step of 8-bit codes is 6 KB for eight MFMAs (256 clocks), 96 B/clk for the four waves where
// a compute unit's L1 delivers 64.  Narrower forms load less and compute more: 1.5 - 6.5 operations per operand dword,
// three dwords per MFMA.
// Measured (fp16 output, one launch inside a graph; before: the general XOR/popcount kernel): W8A8 512 x 4096 x 4096
// 3350 -> 15.3 us, 2048 x 4096 x 4096 40 us, 2048 x 11008 x 4096 112 us (1.65 POP/s); W4A8 15.1 / 41 / 113 us (13.3 / 37 /
// 101 us while 4-bit weights were plane groups: a word of fields takes more operations to unfold than a pair group to cut);
// W8A4 14.4 / 39 / 111 us; W6A6 21 / 63 / 184 us (bound by forming the bytes).  A variant with both operands expanded through LDS (64 x 128
// and 128 x 256 tiles, eight waves, one barrier per k block) took 24.3 and 129 us for W8A8 at the first and third size:
// the chain barrier, LDS read, MFMA, LDS write of every k block was not covered.
#pragma once
#include <hip/hip_ext.h>

#include "apmm_i8_expand.h"
#include "apmm_mfma_common.h"

namespace apmm {
namespace i8 {

using mfma::static_for;
using mfma::vec_word;
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

// slot of load i of half KK
template <int FORM, int KK>
__device__ __forceinline__ int load_slot(const Operand &o, int i)
{
    if (FORM == 1) return 0;
    if (FORM == 2) return KK;
    if (FORM == 3) return i == 0 ? KK : 2;
    if (FORM == 4) return 2 * KK + i;
    if (FORM == kFields) return 3 * KK + i;
    if (FORM == kNibbles) return i < 2 ? 2 * KK + i : i == 2 ? o.pair_slot + KK : o.single_slot;
    return 4 * KK + i;
}

// dword D = 2 tt + jh of operand chunk I = 2 e + tp of half KK
template <int FORM, int KK, int I, int D, int NL>
__device__ __forceinline__ int operand_dword(const Operand &o, const uint4 (&raw)[NL])
{
    constexpr int e = I / 2, tp = I % 2, tt = D / 2, jh = D % 2, t = 2 * tp + tt, ks = 2 * KK + e;
    constexpr int pair_at = 4 * jh + 2 * tt, single_at = 4 * jh + ks;
    if constexpr (FORM == 1) {
        return (int)((vec_word<t>(raw[0]) >> single_at) & 0x01010101u);
    } else if constexpr (FORM == 2) {
        return (int)((vec_word<2 * e + tp>(raw[0]) >> pair_at) & 0x03030303u);
    } else if constexpr (FORM == 3) {
        return (int)folded_dword<3, tp, tt, jh>(vec_word<2 * e>(raw[0]), vec_word<2 * e + 1>(raw[0]), vec_word<ks>(raw[1]), 0u);
    } else if constexpr (FORM == 4) {
        return (int)folded_dword<4, tp, tt, jh>(raw[e].x, raw[e].y, raw[e].z, raw[e].w);
    } else if constexpr (FORM == kFields) {
        constexpr int w = 6 * e + 3 * tp;  // first of the three words of (e, tp)
        auto word = [&](auto i_c) __attribute__((always_inline)) {
            constexpr int i = decltype(i_c)::value;
            return vec_word<i & 3>(raw[i >> 2]);
        };
        const uint32_t w0 = word(std::integral_constant<int, w>{}), w1 = word(std::integral_constant<int, w + 1>{}),
                       w2 = word(std::integral_constant<int, w + 2>{});
        return (int)field_dword<tt, jh>(w0, w1, w2);
    } else if constexpr (FORM == kNibbles) {
        uint32_t v = (vec_word<t>(raw[e]) >> (4 * jh)) & 0x0f0f0f0fu;
        v |= shifted<pair_at - 4>(vec_word<2 * e + tp>(raw[2])) & o.pair_mask;
        v |= ((vec_word<t>(raw[3]) >> single_at) & o.single_mask) << o.single_pos;
        return (int)v;
    } else {
        return (int)vec_word<D>(raw[I]);
    }
}

constexpr int kWM = 2, kWN = 4;  // blocks of a wave tile
constexpr int ksplit_lds_bytes() { return kWM * kWN * 3 * 4 * 64 * 16; }

template <int FA, int FB, bool KSPLIT>
__global__ __launch_bounds__(256) void gemm_mfma_i8_kernel(const uint32_t *a_arg, const uint32_t *w_arg, int32_t *ci_arg,
                                                           uint16_t *cf_arg, int m_arg, int n_arg, int k_arg, uint32_t part_magic,
                                                           int tiles_n, int tiles_m_xn, const uint16_t *ws_arg,
                                                           const uint16_t *as_arg, int p, int q, bool stream)
{
    extern __shared__ __align__(16) int4 red[];  // KSPLIT: [block][partial 0..2][register quad 0..3][lane]
    constexpr int LA = form_loads(FA), LB = form_loads(FB);
    constexpr bool EXPAND_A = FA != kBytes, EXPAND_B = FB != kBytes;
    constexpr int BM = (KSPLIT ? 1 : 2) * 32 * kWM, BN = (KSPLIT ? 1 : 2) * 32 * kWN;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r32 = lane & 31, kh = lane >> 5;
    // XCD-aware tile map: the tile grid in 8 / xn x xn parts, one per XCD, walked down their columns
    // (The way to the first request is scalar arithmetic in 32 bits: 2048 x 4096 x 4096 W8A8 44.0 -> 42.8 us, 300 x 5003 x 3001 W7A5 both 22.1 -> 21.3.  Code sums and
    // scales asked for there as well, 40 loads between the first two stages, cost 3 - 18 %: they are asked for at the end.)
    const uint32_t tiles_m = tiles_m_xn & 0x0fffffff, xn_log = (uint32_t)tiles_m_xn >> 28;
    const uint32_t xcd = blockIdx.x & 7, idx = blockIdx.x >> 3;
    const uint32_t part_m = (tiles_m + (8 >> xn_log) - 1) >> (3 - xn_log), part_n = (tiles_n + (1 << xn_log) - 1) >> xn_log;
    const uint32_t row_of_parts = mfma::quotient(idx, part_m, part_magic);
    const uint32_t tm = (xcd >> xn_log) * part_m + idx - row_of_parts * part_m, tn = (xcd & ((1 << xn_log) - 1)) * part_n + row_of_parts;
    if (tm >= tiles_m || tn >= (uint32_t)tiles_n) return;  // the grid is padded to 8 equal parts
    const int64_t M = m_arg, N = n_arg;
    const int64_t m0 = (int64_t)tm * BM + (KSPLIT ? 0 : (wave >> 1) * 32 * kWM);
    const int64_t n0 = (int64_t)tn * BN + (KSPLIT ? 0 : (wave & 1) * 32 * kWN);
    const uint32_t nrb_a = ((uint32_t)m_arg + 31) / 32, nrb_b = ((uint32_t)n_arg + 31) / 32;
    const int nkb = (int)mfma::padded_k_blocks(k_arg);
    const Operand oa = make_operand<FA>(p), ob = make_operand<FB>(q);

    // this wave's stages: pairs of k blocks, two stages each
    const int pairs = nkb / 2;
    const int p_begin = KSPLIT ? wave * (pairs / 4) + (wave < pairs % 4 ? wave : pairs % 4) : 0;
    const int p_end = KSPLIT ? p_begin + pairs / 4 + (wave < pairs % 4 ? 1 : 0) : pairs;

    constexpr int kSlotBytes = kPlaneWords * 4;
    const uint32_t voff_a = (uint32_t)(kh * oa.slots * kSlotBytes + r32 * 16), voff_b = (uint32_t)(kh * ob.slots * kSlotBytes + r32 * 16);
    const char *pa_blk[kWM], *pb_blk[kWN];
#pragma unroll
    for (int bi = 0; bi < kWM; ++bi) {
        const uint32_t rb = min((uint32_t)(m0 / 32) + bi, nrb_a - 1);  // blocks past the operand: read the last one, never stored
        pa_blk[bi] = reinterpret_cast<const char *>(a_arg) + (uint64_t)(rb * (uint32_t)nkb) * (oa.slots * kSlotBytes);
    }
#pragma unroll
    for (int bj = 0; bj < kWN; ++bj) {
        const uint32_t rb = min((uint32_t)(n0 / 32) + bj, nrb_b - 1);
        pb_blk[bj] = reinterpret_cast<const char *>(w_arg) + (uint64_t)(rb * (uint32_t)nkb) * (ob.slots * kSlotBytes);
    }

    v16i acc[kWM][kWN];
    uint4 ra[2][kWM][LA], rb[2][kWN][LB];  // raw words by stage parity (= half kk)
    v4i af[2][kWM], bf[2][kWN];            // operand chunks by k step parity
    auto load_stage = [&](auto kk_c, int pair) __attribute__((always_inline)) {
        constexpr int kk = decltype(kk_c)::value;
#pragma unroll
        for (int bi = 0; bi < kWM; ++bi)
#pragma unroll
            for (int i = 0; i < LA; ++i)
                ra[kk][bi][i] = *reinterpret_cast<const uint4 *>(pa_blk[bi] + ((int64_t)pair * 2 * oa.slots + load_slot<FA, kk>(oa, i)) * kSlotBytes + voff_a);
#pragma unroll
        for (int bj = 0; bj < kWN; ++bj)
#pragma unroll
            for (int i = 0; i < LB; ++i)
                rb[kk][bj][i] = *reinterpret_cast<const uint4 *>(pb_blk[bj] + ((int64_t)pair * 2 * ob.slots + load_slot<FB, kk>(ob, i)) * kSlotBytes + voff_b);
    };
    constexpr int FRAG0 = EXPAND_A ? 0 : kWM, FRAGS = EXPAND_B ? kWM + kWN : kWM;  // fragments that need forming
    constexpr int TASKS = FRAGS > FRAG0 ? 4 * (FRAGS - FRAG0) : 0, TPM = (TASKS + kWM * kWN - 1) / (kWM * kWN);
    auto form = [&](auto kk_c, auto i_c, auto f_c, auto d_c) __attribute__((always_inline)) {
        constexpr int kk = decltype(kk_c)::value, i = decltype(i_c)::value, f = decltype(f_c)::value, d = decltype(d_c)::value;
        if constexpr (f < kWM) af[i & 1][f][d] = operand_dword<FA, kk, i, d>(oa, ra[kk][f]);
        else bf[i & 1][f - kWM][d] = operand_dword<FB, kk, i, d>(ob, rb[kk][f - kWM]);
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    auto stage = [&](auto kk_c, int next_pair) __attribute__((always_inline)) {
        constexpr int kk = decltype(kk_c)::value;
        using Other = std::integral_constant<int, kk ^ 1>;
        load_stage(Other{}, next_pair);
        __builtin_amdgcn_sched_barrier(0);
        static_for<4 * kWM * kWN>([&](auto x_c) __attribute__((always_inline)) {
            constexpr int x = decltype(x_c)::value, i = x / (kWM * kWN), j = x % (kWM * kWN), bi = j / kWN, bj = j % kWN;
            v4i a, b;
            if constexpr (EXPAND_A) a = af[i & 1][bi];
            else a = v4i{(int)ra[kk][bi][i % LA].x, (int)ra[kk][bi][i % LA].y, (int)ra[kk][bi][i % LA].z, (int)ra[kk][bi][i % LA].w};
            if constexpr (EXPAND_B) b = bf[i & 1][bj];
            else b = v4i{(int)rb[kk][bj][i % LB].x, (int)rb[kk][bj][i % LB].y, (int)rb[kk][bj][i % LB].z, (int)rb[kk][bj][i % LB].w};
            acc[bi][bj] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, acc[bi][bj], 0, 0, 0);
            static_for<TPM>([&](auto t_c) __attribute__((always_inline)) {
                constexpr int task = j * TPM + decltype(t_c)::value;
                if constexpr (task < TASKS) {
                    using F = std::integral_constant<int, FRAG0 + task / 4>;
                    using D = std::integral_constant<int, task % 4>;
                    if constexpr (i + 1 < 4) form(kk_c, std::integral_constant<int, i + 1>{}, F{}, D{});
                    else form(Other{}, I0{}, F{}, D{});
                }
            });
            __builtin_amdgcn_sched_barrier(0);
        });
    };

    if (p_begin < p_end) load_stage(I0{}, p_begin);
#pragma unroll
    for (int bi = 0; bi < kWM; ++bi)
#pragma unroll
        for (int bj = 0; bj < kWN; ++bj)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[bi][bj][v] = 0;
    if (p_begin < p_end) {
        static_for<(FRAGS > FRAG0 ? FRAGS - FRAG0 : 0)>([&](auto f_c) __attribute__((always_inline)) {
            using F = std::integral_constant<int, FRAG0 + decltype(f_c)::value>;
            static_for<4>([&](auto d_c) __attribute__((always_inline)) { form(I0{}, I0{}, F{}, d_c); });
        });
        for (int pair = p_begin; pair < p_end; ++pair) {
            stage(I0{}, pair);                                    // requests the second half of the pair
            stage(I1{}, pair + 1 < p_end ? pair + 1 : pair);      // (the surplus request of the last stage is discarded)
        }
    }

    // ---- recovery and store ----
    const uint32_t ca = value_offset(p), cw = value_offset(q), k_pad = (uint32_t)nkb * kKBlock;
    const uint32_t full = k_pad * ca * cw - (k_pad - (uint32_t)k_arg) * ((1u << p) - 1u) * ((1u << q) - 1u);
    const int32_t *a_sum = reinterpret_cast<const int32_t *>(a_arg) + (uint64_t)(nrb_a * (uint32_t)nkb) * (uint32_t)(kRowBlock * 4 * oa.slots);
    const int32_t *w_sum = reinterpret_cast<const int32_t *>(w_arg) + (uint64_t)(nrb_b * (uint32_t)nkb) * (uint32_t)(kRowBlock * 4 * ob.slots);
    // a missing scale vector reads code sums instead, so that every load is unconditional
    const uint16_t *sa_src = as_arg ? as_arg : reinterpret_cast<const uint16_t *>(a_sum);
    const uint16_t *sw_src = ws_arg ? ws_arg : reinterpret_cast<const uint16_t *>(w_sum);
    uint32_t pa[16], sa_bits[16], pw[kWN], sw_bits[kWN];
    auto request_rows = [&](uint32_t mb) __attribute__((always_inline)) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const uint32_t m = min(mb + 8 * (v / 4) + 4 * kh + (v % 4), (uint32_t)m_arg - 1);  // row of register v
            pa[v] = (uint32_t)a_sum[m];
            sa_bits[v] = sa_src[m];
        }
    };
#pragma unroll
    for (int bj = 0; bj < kWN; ++bj) {
        const uint32_t n = min((uint32_t)n0 + 32 * bj + r32, (uint32_t)n_arg - 1);
        pw[bj] = (uint32_t)w_sum[n];
        sw_bits[bj] = sw_src[n];
    }
    const bool pair_ok = (N & 1) == 0 && (reinterpret_cast<uintptr_t>(cf_arg) & 3u) == 0;
    // one 32 x 32 block, inner ones with streaming stores by the launcher's rule
    auto store_block = [&](const v16i &s, int64_t mb, auto bj_c) __attribute__((always_inline)) {
        constexpr int bj = decltype(bj_c)::value;
        const int64_t n = n0 + 32 * bj + r32;
        const bool interior = mb + 32 <= M && n0 + 32 * bj + 32 <= N;
        const uint32_t ct = full - 2u * ca * (pw[bj] - code_bias(q) * k_pad);
        const float sw = half_bits_to_float((uint16_t)(ws_arg ? sw_bits[bj] : 0x3c00u));
        int32_t c[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) c[v] = (int32_t)(4u * (uint32_t)s[v] + ct - 2u * cw * (pa[v] - code_bias(p) * k_pad));
        auto row = [&](int v) __attribute__((always_inline)) { return mb + 8 * (v / 4) + 4 * kh + (v % 4); };
        auto sa = [&](int v) __attribute__((always_inline)) { return half_bits_to_float((uint16_t)(as_arg ? sa_bits[v] : 0x3c00u)); };
        if (ci_arg) {
            if (interior && stream) {
                edge_of_streaming();
#pragma unroll
                for (int v = 0; v < 16; ++v) __builtin_nontemporal_store(c[v], ci_arg + row(v) * N + n);
                edge_of_streaming();
            } else if (interior) {
#pragma unroll
                for (int v = 0; v < 16; ++v) ci_arg[row(v) * N + n] = c[v];
            } else {
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    if (row(v) < M && n < N) ci_arg[row(v) * N + n] = c[v];
            }
        }
        if (cf_arg && interior && pair_ok) {
            // rows in pairs: the even lane of a lane pair stores both columns of the first row, the odd lane both of the second
            const bool odd = lane & 1;
            const uint32_t selector = swap_pair_selector(odd);
            uint32_t word[8];
#pragma unroll
            for (int v = 0; v < 16; v += 2) {
                word[v / 2] = swap_pair(half_pair((float)c[v] * sa(v), (float)c[v + 1] * sa(v + 1), sw), selector);
            }
            auto dst = [&](int i) __attribute__((always_inline)) {
                return reinterpret_cast<uint32_t *>(cf_arg + (row(2 * i) + (odd ? 1 : 0)) * N + n - (odd ? 1 : 0));
            };
            if (stream) {
                edge_of_streaming();
#pragma unroll
                for (int i = 0; i < 8; ++i) __builtin_nontemporal_store(word[i], dst(i));
                edge_of_streaming();
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i) *dst(i) = word[i];
            }
        } else if (cf_arg) {
#pragma unroll
            for (int v = 0; v < 16; ++v)
                if (row(v) < M && n < N) cf_arg[row(v) * N + n] = float_to_half_bits((float)c[v] * sa(v) * sw);
        }
    };
    if constexpr (KSPLIT) {
        // the partial tiles meet: wave w finishes blocks 2 (w % 2), + 1 of row block w / 2
        request_rows((uint32_t)m0 + 32 * (wave >> 1));
        static_for<kWM * kWN>([&](auto b_c) __attribute__((always_inline)) {
            constexpr int b = decltype(b_c)::value, bi = b / kWN, bj = b % kWN, own = 2 * bi + bj / 2;
            if (wave != own) {
                int4 *dst = red + (b * 3 + ((wave - own + 4) & 3) - 1) * 256 + lane;
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4)
                    dst[q4 * 64] = make_int4(acc[bi][bj][4 * q4], acc[bi][bj][4 * q4 + 1], acc[bi][bj][4 * q4 + 2], acc[bi][bj][4 * q4 + 3]);
            }
        });
        __syncthreads();
        static_for<kWM * kWN>([&](auto b_c) __attribute__((always_inline)) {
            constexpr int b = decltype(b_c)::value, bi = b / kWN, bj = b % kWN, own = 2 * bi + bj / 2;
            if (wave != own) return;
            int4 t[12];  // all twelve reads in flight before the first add
#pragma unroll
            for (int i = 0; i < 12; ++i) t[i] = red[(b * 3 + i / 4) * 256 + (i % 4) * 64 + lane];
            __builtin_amdgcn_sched_barrier(0);
            v16i s = acc[bi][bj];
#pragma unroll
            for (int i = 0; i < 12; ++i) {
                s[4 * (i % 4)] += t[i].x; s[4 * (i % 4) + 1] += t[i].y; s[4 * (i % 4) + 2] += t[i].z; s[4 * (i % 4) + 3] += t[i].w;
            }
            store_block(s, m0 + 32 * bi, std::integral_constant<int, bj>{});
        });
    } else {
        static_for<kWM>([&](auto bi_c) __attribute__((always_inline)) {
            constexpr int bi = decltype(bi_c)::value;
            request_rows((uint32_t)m0 + 32 * bi);
            __builtin_amdgcn_sched_barrier(0);
            static_for<kWN>([&](auto bj_c) __attribute__((always_inline)) { store_block(acc[bi][decltype(bj_c)::value], m0 + 32 * bi, bj_c); });
        });
    }
}

template <int FA, int FB, bool KSPLIT>
hipError_t launch_variant(const GemmArgs &g, hipStream_t stream)
{
    constexpr int BM = (KSPLIT ? 1 : 2) * 32 * kWM, BN = (KSPLIT ? 1 : 2) * 32 * kWN, lds = KSPLIT ? ksplit_lds_bytes() : 0;
    const int64_t tiles_m = (g.M + BM - 1) / BM, tiles_n = (g.N + BN - 1) / BN;
    if (tiles_m >= (1 << 28) || tiles_n >= (1 << 28) || g.M > 0x7fffffffLL || g.N > 0x7fffffffLL || g.K > 0x7fffffffLL) return hipErrorInvalidValue;
    // parts of the tile grid per XCD: the cut that leaves an XCD the fewest packed bytes to read
    int xn_log = 0;
    double best = 0;
    for (int l = 0; l <= 3; ++l) {
        const int64_t pm = (tiles_m + (8 >> l) - 1) / (8 >> l), pn = (tiles_n + (1 << l) - 1) / (1 << l);
        const double bytes = (double)pm * BM * activation_slots(g.p) + (double)pn * BN * g.q;
        if (l == 0 || bytes < best) { best = bytes; xn_log = l; }
    }
    const int64_t part_m = (tiles_m + (8 >> xn_log) - 1) / (8 >> xn_log), part_n = (tiles_n + (1 << xn_log) - 1) / (1 << xn_log);
    const int64_t grid = 8 * part_m * part_n;
    if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
    const int tiles_m_xn = (int)tiles_m | (xn_log << 28);
    const uint32_t magic = mfma::divisor_magic(part_m, part_m * part_n);
    // Streaming stores where the rows are whole lines (W8A8 2048 x 11008 x 4096 both 156 -> 119 us).  Rows of parts of lines: int32 up to 22 MB
    // of outputs, whole tiles also before an fp16 output (both outputs of the K split 0.94 - 0.97 of the streaming time at 10 - 18 MB, fp16
    // alone 0.97 up to 3 MB and 0.85 at 30).
    const mfma::OutputRows rows(g);
    const bool streaming = rows.whole || (g.c_i32 && (KSPLIT ? !g.c_f16 : rows.up_to_l2(22000000)));
    auto kernel = gemm_mfma_i8_kernel<FA, FB, KSPLIT>;
    if constexpr (KSPLIT) {
        static thread_local int prepared_device = -1;  // the LDS limit is a per-device attribute of the function
        int dev = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return e;
        if (prepared_device != dev) {
            e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
            if (e != hipSuccess) return e;
            prepared_device = dev;
        }
    }
    const KernelTiming timing = take_kernel_timing();
    note_kernel("gemm_mfma_i8_kernel<%d,%d,%s>", g.p, g.q, KSPLIT ? "ksplit" : "tiles");
    const dim3 blocks((unsigned)grid), threads(256);
    if (timing.start || timing.stop)
        hipExtLaunchKernelGGL(kernel, blocks, threads, lds, stream, timing.start, timing.stop, 0, g.a, g.w, g.c_i32, g.c_f16, (int)g.M,
                              (int)g.N, (int)g.K, magic, (int)tiles_n, tiles_m_xn, g.w_scale, g.a_scale, g.p, g.q, streaming);
    else
        hipLaunchKernelGGL(kernel, blocks, threads, lds, stream, g.a, g.w, g.c_i32, g.c_f16, (int)g.M, (int)g.N, (int)g.K, magic,
                           (int)tiles_n, tiles_m_xn, g.w_scale, g.a_scale, g.p, g.q, streaming);
    return hipGetLastError();
}

template <int FA, int FB>
hipError_t launch_forms(const GemmArgs &g, hipStream_t stream, bool ksplit)
{
    return ksplit ? launch_variant<FA, FB, true>(g, stream) : launch_variant<FA, FB, false>(g, stream);
}

}  // namespace i8
}  // namespace apmm
