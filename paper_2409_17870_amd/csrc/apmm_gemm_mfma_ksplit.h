// Design A for outputs too small to give every compute unit a large tile: the four waves of a workgroup split K.
//
// The algebra is that of apmm_gemm_mfma_direct.h (paper Sec. 3.2: the shift-and-add over plane pairs, moved in
// front of the multiplier; recovery terms as the accumulator's start value).  What differs is who shares what.
// There the four waves of a workgroup own four parts of the output tile and each sweeps all of K, so that two
// waves load (and expand) every packed fragment; the tiles that fit the register file then ask the L1 of a compute
// unit for more bytes per MFMA than it delivers, most of all with activations in the 6-bit field form, and a
// prefill of a few hundred tokens leaves a third of the chip without a tile.  Here every wave owns the WHOLE
// workgroup tile (WM x WN blocks of 32 x 32, as many as the accumulator registers hold) and a quarter of the
// stages of K (paper Sec. 4.2 item 2 partitions K in time; this partitions it across waves as well): no fragment
// is loaded twice inside a compute unit, the bytes per MFMA are those of the largest wave tile, and a 512 x 5120
// output is 256 tiles of 64 x 160 instead of 160 of 128 x 128.  The four partial tiles meet in LDS once, at the
// end: every wave writes the blocks it does not own, and after one barrier adds the three other partials of the
// blocks it owns (fp32 sums of integers below 2^24: exact in any order) and stores them.  The recovery terms
// start the accumulators of wave 0 only.
#pragma once
#include <hip/hip_ext.h>

#include "apmm_gemm_mfma_lds.h"

namespace apmm {
namespace mfma {

// Owner (wave) of block (bi, bj) of the workgroup tile in the final reduction: every wave's blocks lie in one
// row block, so that it needs one set of token scales.
constexpr int ksplit_owner(int wm, int wn, int bi, int bj)
{
    return wm == 1 ? bj * 4 / wn : wm == 2 ? 2 * bi + (bj >= (wn + 1) / 2 ? 1 : 0) : bi;
}
// The 128 x 128 tile (4 x 4 blocks, 256 accumulators per wave): stages of half a k block, for which the raw words of two
// stages fit beside the accumulators, and the partial tiles meet in two rounds of half the column blocks.  10 KB per k step
// of 16 MFMAs (W4A4), where four wave tiles of 64 x 64 ask L1 for 20: half the time per k, for 6 us more at the end.
constexpr bool ksplit_half(int wm, int wn) { return wm * wn > 12; }
constexpr int ksplit_rounds(int wm, int wn) { return ksplit_half(wm, wn) ? 2 : 1; }
constexpr int ksplit_lds_bytes(int wm, int wn) { return wm * wn / ksplit_rounds(wm, wn) * (ksplit_half(wm, wn) ? 4 : 3) * 4 * 64 * 16; }

// Streaming stores, also when both outputs are written (512 x 5120 x 5120 W2A4 16.7 -> 13.3 us, 512 x 4096 x 4096 W2A2 10.7 -> 9.1, 203 x 4096 x
// 4096 7.2 -> 6.8).  Plain ones for both outputs with rows of parts of lines, up to 8 MB (128 x 4098 x 512 W2A2 4.9 against 5.1 us) and in the
// 128 x 128 tile in registers (2048 x 1500 x 11008 W4A2 24.0 / 27.9).  Not in the tiles of 160 and 192 columns, whose outputs are larger than
// that: one more form of the store of every block makes 67 KB of code 80 (512 x 5120 x 11008 W4A4 both 4 - 6 % slower).
constexpr bool ksplit_always_streams(int wm, int wn) { return wm * wn > 8 && !ksplit_half(wm, wn); }
inline bool ksplit_streams(int wm, int wn, const GemmArgs &g)
{
    const OutputRows rows(g);
    return ksplit_always_streams(wm, wn) || !rows.both || rows.whole || (!ksplit_half(wm, wn) && rows.fit_l2());
}

template <int P, int Q, int WM, int WN>
__device__ __forceinline__ void ksplit_tile(float4 *red, const uint32_t *a_arg, const uint32_t *w_arg, int32_t *ci_arg, uint16_t *cf_arg, int m_arg, int n_arg,
                                            int k_arg, uint32_t part_magic, int tiles_n, int tiles_m_xn, const uint16_t *ws_arg, const uint16_t *as_arg,
                                            bool stream)
{
    // red: [block][partial 0..2][register quad 0..3][lane]
    static_assert(P >= 1 && P <= 4 && Q >= 1 && Q <= 4, "instantiated for codes of up to four bits");
    static_assert(WM == 1 || WM == 2 || WM == 4, "row blocks per tile");
    static_assert(ksplit_lds_bytes(WM, WN) <= 160 * 1024, "the partial copies of every block of a round must fit the LDS");
    constexpr bool AF = activation_field_form(P);
    constexpr int SLOTS_A = activation_slots(P);
    constexpr int NB = WM * WN;
    constexpr bool HALF = ksplit_half(WM, WN);
    constexpr int KS = HALF ? 2 : 4;  // MFMA k steps per stage
    // The 64 x 64 tile with 6-bit fields against folded weights: 248 of the 256 registers of a wave hold accumulators, raw words
    // and fragments.  The lane's offset is hidden from the compiler at each use there, so that the addresses stay a scalar
    // base and one offset register; as 64-bit vector pointers they were spilled and fetched back inside the k loop, each
    // behind a wait for all loads in flight (W4A4, 65 x 4096 x 4096 8.3 -> 6.7 us, 256 x 4096 x 11008 16.7 -> 13.4 us; W3A3 256 x
    // 4096 x 4096 7.9 -> 7.4 us, 256 x 4096 x 11008 13.3 -> 12.9 us.  Half stages as in the 128 x 128 tile take 6.4 and 15.3,
    // 7.8 and 15.3 us, one workgroup to a compute unit 7.3 and 16.9, 7.6 and 13.0 us).
    constexpr bool TIGHT = WM * WN == 4 && AF && Q > 2;
    auto hidden = [](uint32_t v) __attribute__((always_inline)) { return TIGHT ? use_here(v) : v; };
    constexpr int LOADS_A = HALF ? half_slots(P, AF) : SLOTS_A, LOADS_B = HALF ? half_slots(Q, false) : Q;
    // Fields: the slot that two k steps share is copied by hand, a step ahead.  Left to itself the compiler copies it right behind the
    // loads of a stage, in every second stage, and waits there for all of them.  512 x 5120 x 5120 W2A4 13.1 -> 12.6 us, W4A4 15.9 -> 15.2,
    // W3A3 15.7 -> 14.6, 512 x 5120 x 13824 W2A4 24.0 -> 23.1.  (The 64 x 64 tile with 4-bit weights has no registers for the copies,
    // the 128 x 128 tile is not faster.)
    constexpr bool MID = AF && !HALF && !(WM * WN == 4 && Q == 4);
    constexpr uint32_t ca = (1u << P) - 1, cw = (1u << Q) - 1;
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r32 = lane & 31, kh = lane >> 5;
    // Workgroups are dealt round-robin to the 8 XCDs, each with an L2 of its own.  The tile grid is cut into
    // 8 / xn x xn parts, one per XCD, and a part is walked down its columns: the workgroups that run together on an
    // XCD share the packed rows of a few column tiles and of the part's row tiles (tiles_m_xn = tiles_m | log2(xn) << 28).
    // (The way to the first request is scalar arithmetic in 32 bits, 145 instead of 215 instructions for 64 x 160: 203 x 4096 x 4096 W2A2 6.6 -> 6.25 us, 300 x
    // 2000 x 700 W2A3 5.7 -> 5.3, 1024 x 4096 x 11008 W4A4 33.7 -> 32.8.)
    const uint32_t tiles_m = tiles_m_xn & 0x0fffffff, xn_log = (uint32_t)tiles_m_xn >> 28;
    const uint32_t xcd = blockIdx.x & 7, idx = blockIdx.x >> 3;
    const uint32_t part_m = (tiles_m + (8 >> xn_log) - 1) >> (3 - xn_log), part_n = (tiles_n + (1 << xn_log) - 1) >> xn_log;
    const uint32_t row_of_parts = quotient(idx, part_m, part_magic);
    const uint32_t tm = (xcd >> xn_log) * part_m + idx - row_of_parts * part_m, tn = (xcd & ((1 << xn_log) - 1)) * part_n + row_of_parts;
    if (tm >= tiles_m || tn >= (uint32_t)tiles_n) return;  // the grid is padded to 8 equal parts
    const int64_t M = m_arg, N = n_arg;
    const int64_t m0 = (int64_t)tm * (32 * WM), n0 = (int64_t)tn * (32 * WN);
    const uint32_t nkb = padded_k_blocks(k_arg), nrb_a = ((uint32_t)m_arg + 31) / 32, nrb_b = ((uint32_t)n_arg + 31) / 32;

    // this wave's stages of K: nst stages of two k blocks, dealt as evenly as they go
    const uint32_t nst = nkb / 2;
    const int s_begin = wave * (nst / 4) + min((uint32_t)wave, nst % 4);
    const int s_count = nst / 4 + ((uint32_t)wave < nst % 4 ? 1 : 0);
    const int s_end = s_begin + s_count;

    // Addresses: a uniform pointer per block (row blocks past the operand read the last one; never stored) plus
    // one lane offset per operand: row r32 of k block kh of a stage.
    constexpr int kSlotBytes = kPlaneWords * 4;
    constexpr int kStageBytesA = 2 * SLOTS_A * kSlotBytes, kStageBytesB = 2 * Q * kSlotBytes;
    const uint32_t voff_a = (uint32_t)(kh * SLOTS_A * kSlotBytes + r32 * 16);
    const uint32_t voff_b = (uint32_t)(kh * Q * kSlotBytes + r32 * 16);
    const char *pa_blk[WM], *pb_blk[WN];
#pragma unroll
    for (int bi = 0; bi < WM; ++bi) {
        const uint32_t rb = min(tm * WM + bi, nrb_a - 1);
        pa_blk[bi] = reinterpret_cast<const char *>(a_arg) + (uint64_t)(rb * nkb) * (SLOTS_A * kSlotBytes);
    }
#pragma unroll
    for (int bj = 0; bj < WN; ++bj) {
        const uint32_t rb = min(tn * WN + bj, nrb_b - 1);
        pb_blk[bj] = reinterpret_cast<const char *>(w_arg) + (uint64_t)(rb * nkb) * (Q * kSlotBytes);
    }

    v16f acc[WM][WN];
    uint4 ra[2][WM][LOADS_A], rb[2][WN][LOADS_B];  // raw words of a stage, by stage parity (HALF: by half of the k block)
    v4i af[2][AF ? 1 : WM];                  // formed fragments, by k step parity
    uint2 am[2][MID ? WM : 1];               // fields: the words of an operand that share a slot with the neighbouring k step
    OperandFrag<Q> bf[2][WN];

    auto load_stage = [&](auto buf_c, int st) __attribute__((always_inline)) {
        constexpr int buf = decltype(buf_c)::value;
#pragma unroll
        for (int bi = 0; bi < WM; ++bi) {
            const char *src = pa_blk[bi] + (int64_t)st * kStageBytesA + hidden(voff_a);
#pragma unroll
            for (int i = 0; i < LOADS_A; ++i)
                ra[buf][bi][i] = *reinterpret_cast<const uint4 *>(src + (HALF ? half_slot(P, AF, buf, i) : i) * kSlotBytes);
        }
#pragma unroll
        for (int bj = 0; bj < WN; ++bj) {
            const char *src = pb_blk[bj] + (int64_t)st * kStageBytesB + hidden(voff_b);
#pragma unroll
            for (int i = 0; i < LOADS_B; ++i)
                rb[buf][bj][i] = *reinterpret_cast<const uint4 *>(src + (HALF ? half_slot(Q, false, buf, i) : i) * kSlotBytes);
        }
    };

    // First requests: the wave's first stage, then the code sums (wave 0 seeds the
    // accumulators with the recovery terms, the others start at zero).
    if (s_count > 0) load_stage(I0{}, s_begin);
    {
        const int32_t *a_sum = reinterpret_cast<const int32_t *>(a_arg) + (uint64_t)(nrb_a * nkb) * (kRowBlock * SLOTS_A * 4);
        const int32_t *w_sum = reinterpret_cast<const int32_t *>(w_arg) + (uint64_t)(nrb_b * nkb) * (kRowBlock * Q * 4);
        float a_init[WM], b_init[WN];
#pragma unroll
        for (int bj = 0; bj < WN; ++bj) {
            const uint32_t n = min((tn * WN + bj) * 32 + r32, nrb_b * 32 - 1);
            const float ct = (float)(int32_t)((uint32_t)k_arg * ca * cw - 2u * ca * (uint32_t)w_sum[n]);
            b_init[bj] = wave != 0 ? 0.f : kh == 0 ? 1.0f : ct;
        }
#pragma unroll
        for (int bi = 0; bi < WM; ++bi) {
            const uint32_t m = min((tm * WM + bi) * 32 + r32, nrb_a * 32 - 1);
            const float rt = -(float)(2u * cw * (uint32_t)a_sum[m]);
            a_init[bi] = wave != 0 ? 0.f : kh == 0 ? rt : 1.0f;
        }
        v16f zero;
#pragma unroll
        for (int v = 0; v < 16; ++v) zero[v] = 0.f;
#pragma unroll
        for (int bi = 0; bi < WM; ++bi)
#pragma unroll
            for (int bj = 0; bj < WN; ++bj)
                acc[bi][bj] = __builtin_amdgcn_mfma_f32_32x32x2f32(a_init[bi], b_init[bj], zero, 0, 0, 0);
    }

    // This wave's stages of the sweep of K.
    if (s_count > 0) {
        constexpr int PER_KS = NB;
        constexpr int TASKS_A = (MID ? 2 : AF ? 0 : 4) * WM, DB = operand_dwords(Q);
        constexpr int TASKS = TASKS_A + DB * WN;  // operand dwords to form per k step, A blocks first
        constexpr int TPM = (TASKS + PER_KS - 1) / PER_KS;
        auto form = [&](auto buf_c, auto ks_c, auto task_c) __attribute__((always_inline)) {
            constexpr int buf = decltype(buf_c)::value, ks = decltype(ks_c)::value, task = decltype(task_c)::value;
            if constexpr (task < TASKS_A) {
                constexpr int f = task / (MID ? 2 : 4), d = task % (MID ? 2 : 4);
                if constexpr (MID) {
                    if constexpr (d == 0) am[ks & 1][f].x = copy_here(vec_word<2 * (ks & 1)>(ra[buf][f][3 * (ks / 2) + 1]));
                    else am[ks & 1][f].y = copy_here(vec_word<2 * (ks & 1) + 1>(ra[buf][f][3 * (ks / 2) + 1]));
                } else if constexpr (HALF) af[ks & 1][f][d] = (int)half_operand_dword<P, buf, ks, d>(ra[buf][f]);
                else af[ks & 1][f][d] = (int)operand_dword<P, ks, d>(ra[buf][f]);
            } else {
                constexpr int f = (task - TASKS_A) / DB, d = (task - TASKS_A) % DB;
                if constexpr (HALF) bf[ks & 1][f][d] = (int)half_operand_dword<Q, buf, ks, d>(rb[buf][f]);
                else bf[ks & 1][f][d] = (int)operand_dword<Q, ks, d>(rb[buf][f]);
            }
        };
        auto stage = [&](auto buf_c, int st) __attribute__((always_inline)) {
            constexpr int buf = decltype(buf_c)::value;
            using Other = std::integral_constant<int, buf ^ 1>;
            load_stage(Other{}, (HALF && buf == 0) || st + 1 >= s_end ? st : st + 1);  // the surplus load is discarded
            __builtin_amdgcn_sched_barrier(0);
            static_for<KS * PER_KS>([&](auto i_c) __attribute__((always_inline)) {
                constexpr int i = decltype(i_c)::value;
                constexpr int ks = i / PER_KS, j = i % PER_KS, bi = j / WN, bj = j % WN;
                constexpr int format_a = operand_format(P), format_b = operand_format(Q);
                v8i a8;
                if constexpr (MID) a8 = field_operand<ks>(ra[buf][bi], am[ks & 1][bi]);
                else if constexpr (AF) a8 = field_operand<ks>(ra[buf][bi]);
                else a8 = widen(af[ks & 1][bi]);
                acc[bi][bj] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                    a8, widen(bf[ks & 1][bj]), acc[bi][bj], format_a, format_b, 0, operand_exponent(P, HALF ? 2 * buf + ks : ks), 0,
                    operand_exponent(Q, HALF ? 2 * buf + ks : ks));
                static_for<TPM>([&](auto t_c) __attribute__((always_inline)) {
                    constexpr int task = j * TPM + decltype(t_c)::value;
                    if constexpr (task < TASKS) {
                        using X = std::integral_constant<int, task>;
                        if constexpr (ks + 1 < KS) form(buf_c, std::integral_constant<int, ks + 1>{}, X{});
                        else form(Other{}, I0{}, X{});
                    }
                });
                __builtin_amdgcn_sched_barrier(0);
            });
        };
        static_for<TASKS>([&](auto t_c) __attribute__((always_inline)) { form(I0{}, I0{}, t_c); });
        int st = s_begin;
        if constexpr (HALF) {
            for (; st < s_end; ++st) {
                stage(I0{}, st);
                stage(I1{}, st);
            }
        } else {
            for (; st + 1 < s_end; st += 2) {
                stage(I0{}, st);
                stage(I1{}, st + 1);
            }
            if (st < s_end) stage(I0{}, st);
        }
    }

    using T = std::true_type;
    using F = std::false_type;
    // ---- the four partial tiles meet ----
    // Scales of the blocks this wave will store, requested before the exchange so that they are there after it:
    // the 16 token scales of this lane's rows (all of a wave's blocks lie in row block bi_own), one channel scale
    // per block.
    const int bi_own = WM == 1 ? 0 : WM == 2 ? wave >> 1 : wave;
    const int lane_out = (int)hidden((uint32_t)lane), c32 = lane_out & 31;  // (nothing of the store is kept through the k loop)
    const int64_t m_own = m0 + bi_own * 32 + 4 * (lane_out >> 5);  // row of register v: m_own + 8 (v / 4) + v % 4
    // (Unconditional loads from clamped addresses, one uniform branch around each set: a load under a per-lane
    // condition is followed by a wait, and 26 such waits in a row cost 2 us here.)
    uint32_t sa_bits[16], sw_bits[WN];
#pragma unroll
    for (int v = 0; v < 16; ++v) sa_bits[v] = 0x3c00u;
#pragma unroll
    for (int bj = 0; bj < WN; ++bj) sw_bits[bj] = 0x3c00u;
    if (cf_arg && as_arg) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            sa_bits[v] = as_arg[min((uint32_t)m_own + 8 * (v / 4) + (v % 4), (uint32_t)m_arg - 1)];
        }
    }
    if (cf_arg && ws_arg) {
#pragma unroll
        for (int bj = 0; bj < WN; ++bj) {
            sw_bits[bj] = ws_arg[min((uint32_t)n0 + bj * 32 + c32, (uint32_t)n_arg - 1)];
        }
    }
    // Store of one owned block.  GUARD: border tile, every element tested.  PAIR (interior, even N, 4-byte aligned
    // fp16 output): neighbouring lanes hold neighbouring columns; rows are taken in pairs, the even lane of a lane
    // pair collects both columns of the first row, the odd lane both columns of the second (one lane exchange),
    // and each stores one dword instead of two halves.  NT: streaming stores of inner tiles (rule: ksplit_streams).
    const bool interior = (m0 + 32 * WM <= M) && (n0 + 32 * WN <= N);
    const bool pair_ok = (N & 1) == 0 && (reinterpret_cast<uintptr_t>(cf_arg) & 3u) == 0;
    if constexpr (ksplit_always_streams(WM, WN)) stream = true;
    const bool odd = lane_out & 1;
    const uint32_t selector = swap_pair_selector(odd);
    float sa_f[16];
#pragma unroll
    for (int v = 0; v < 16; ++v) sa_f[v] = half_bits_to_float((uint16_t)use_here(sa_bits[v]));
    // stores the finished block in this wave's row block and the columns from n on
    auto finish = [&](const v16f &c, int64_t n, uint32_t sw_h) __attribute__((always_inline)) {
        auto emit = [&](auto guard_c, auto i32_c, auto f16_c, auto pair_c, auto nt_c) __attribute__((always_inline)) {
            constexpr bool GUARD = decltype(guard_c)::value, I32 = decltype(i32_c)::value, F16 = decltype(f16_c)::value,
                           PAIR = decltype(pair_c)::value, NT = decltype(nt_c)::value;
            if constexpr (NT) edge_of_streaming();
            const float sw = half_bits_to_float((uint16_t)use_here(sw_h));
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int64_t m = m_own + 8 * (v / 4) + (v % 4);
                if (GUARD && (m >= M || n >= N)) continue;
                if constexpr (I32) {
                    int32_t *dst = ci_arg + m * N + n;
                    if constexpr (NT) __builtin_nontemporal_store((int32_t)c[v], dst);
                    else *dst = (int32_t)c[v];
                }
                if constexpr (F16 && !PAIR) cf_arg[m * N + n] = float_to_half_bits(c[v] * sa_f[v] * sw);
                if constexpr (F16 && PAIR) {
                    if (v % 2 == 0) {
                        const uint32_t word = swap_pair(half_pair(c[v] * sa_f[v], c[(v + 1) & 15] * sa_f[(v + 1) & 15], sw), selector);
                        // odd lanes write the row below at the column to the left
                        uint32_t *dst = reinterpret_cast<uint32_t *>(cf_arg + (m + (odd ? 1 : 0)) * N + n - (odd ? 1 : 0));
                        if constexpr (NT) __builtin_nontemporal_store(word, dst);
                        else *dst = word;
                    }
                }
            }
            if constexpr (NT) edge_of_streaming();
        };
        if (ci_arg) {
            if (interior && stream) emit(F{}, T{}, F{}, F{}, T{});
            else if (interior) emit(F{}, T{}, F{}, F{}, F{});
            else emit(T{}, T{}, F{}, F{}, F{});
        }
        if (cf_arg) {
            if (interior && pair_ok && stream) emit(F{}, F{}, T{}, T{}, T{});
            else if (interior && pair_ok) emit(F{}, F{}, T{}, T{}, F{});
            else if (interior) emit(F{}, F{}, T{}, F{}, F{});
            else emit(T{}, F{}, T{}, F{}, F{});
        }
    };
    constexpr int ROUNDS = ksplit_rounds(WM, WN), WNR = WN / ROUNDS, NBR = NB / ROUNDS;  // column blocks and blocks of a round
    static_for<ROUNDS>([&](auto round_c) __attribute__((always_inline)) {
        constexpr int round = decltype(round_c)::value;
        if constexpr (round > 0) __syncthreads();  // every wave has read the partials of the round before
        if constexpr (HALF) {
            // The same code for every wave: each block of the round goes to LDS from all four waves and is taken from there by
            // the wave that owns its row block.  With code of its own per block and owner, as for the smaller tiles, the
            // registers spilled and the straight-line code of sixteen blocks was fetched cold: 1024 x 4096 x 4096 W4A4 23.7 ->
            // 16.8 us.  (The smaller tiles are better off without the fourth copy: 65 x 4096 x 4096 W2A2 5.7 against 6.2 us.)
            static_for<NBR>([&](auto b_c) __attribute__((always_inline)) {
                constexpr int b = decltype(b_c)::value, bi = b / WNR, bj = round * WNR + b % WNR;
                float4 *dst = red + (b * 4 + wave) * 256 + lane_out;
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4)
                    dst[q4 * 64] = make_float4(acc[bi][bj][4 * q4], acc[bi][bj][4 * q4 + 1], acc[bi][bj][4 * q4 + 2], acc[bi][bj][4 * q4 + 3]);
            });
            __syncthreads();
#pragma unroll 1
            for (int jj = 0; jj < WNR; ++jj) {
                float4 t[16];
#pragma unroll
                for (int i = 0; i < 16; ++i) t[i] = red[((wave * WNR + jj) * 4 + i / 4) * 256 + (i % 4) * 64 + lane_out];
                v16f c;
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4) {
                    c[4 * q4] = (t[q4].x + t[4 + q4].x) + (t[8 + q4].x + t[12 + q4].x);
                    c[4 * q4 + 1] = (t[q4].y + t[4 + q4].y) + (t[8 + q4].y + t[12 + q4].y);
                    c[4 * q4 + 2] = (t[q4].z + t[4 + q4].z) + (t[8 + q4].z + t[12 + q4].z);
                    c[4 * q4 + 3] = (t[q4].w + t[4 + q4].w) + (t[8 + q4].w + t[12 + q4].w);
                }
                static_assert(WNR == 2 || !HALF, "two column blocks per round");
                finish(c, n0 + (round * WNR + jj) * 32 + c32, jj ? sw_bits[round * WNR + 1] : sw_bits[round * WNR]);
            }
        } else {
            static_for<NBR>([&](auto b_c) __attribute__((always_inline)) {
                constexpr int b = decltype(b_c)::value, bi = b / WN, bj = b % WN;
                constexpr int own = ksplit_owner(WM, WN, bi, bj);
                if (wave != own) {
                    const int part = ((wave - own + 4) & 3) - 1;
                    float4 *dst = red + (b * 3 + part) * 256 + lane_out;
#pragma unroll
                    for (int q4 = 0; q4 < 4; ++q4)
                        dst[q4 * 64] = make_float4(acc[bi][bj][4 * q4], acc[bi][bj][4 * q4 + 1], acc[bi][bj][4 * q4 + 2],
                                                   acc[bi][bj][4 * q4 + 3]);
                }
            });
            __syncthreads();
            static_for<NBR>([&](auto b_c) __attribute__((always_inline)) {
                constexpr int b = decltype(b_c)::value, bi = b / WN, bj = b % WN;
                constexpr int own = ksplit_owner(WM, WN, bi, bj);
                if (wave != own) return;
                // all twelve reads of the three other partials in flight before the first add
                float4 t[12];
#pragma unroll
                for (int i = 0; i < 12; ++i) t[i] = red[(b * 3 + i / 4) * 256 + (i % 4) * 64 + lane_out];
                __builtin_amdgcn_sched_barrier(0);
                v16f c = acc[bi][bj];
#pragma unroll
                for (int i = 0; i < 12; ++i) {
                    c[4 * (i % 4)] += t[i].x; c[4 * (i % 4) + 1] += t[i].y; c[4 * (i % 4) + 2] += t[i].z; c[4 * (i % 4) + 3] += t[i].w;
                }
                finish(c, n0 + bj * 32 + c32, sw_bits[bj]);
            });
        }
    });
}

// The 128 x 128 tile (4 x 4 blocks) in two forms.  Up to K = 9216 (ksplit_lds_max_k), and with 2-bit weights at every K: two groups of four waves, each with half
// of K, that share their operands through LDS (apmm_gemm_mfma_lds.h).  It starts and ends faster and, with twice the waves, waits
// less, but a product needs 1.25 KB of LDS reads (W4A4) where the four waves with 256 accumulators read their words from L1 once for
// sixteen.  Microseconds, LDS / registers: K = 4096, 1024 x 4096 outputs W4A4 14.3 / 16.9, W3A3 14.3 / 16.7, W4A2 12.9 / 15.2; K = 8192 25.2 / 25.8,
// 23.7 / 25.1, 21.2 / 22.0; K = 11008 33.5 / 32.6, 30.8 / 30.9, 27.6 / 27.1; with 2 bits at K = 11008 W2A4 27.9 / 30.0, W2A2 22.0 / 22.6, W2A1
// 20.5 / 21.8.
// With 1- and 2-bit activations the registers catch up earlier, operands and outputs in rotation over seven outputs, LDS / registers: W3A2 fp16 0.97 -
// 1.03 at K = 8704 and 1.00 - 1.05 at 9216, int32 alone 0.99 - 1.03 at 6144, 1.02 - 1.05 at 7168, 1.03 - 1.09 beyond; W4A2 int32 0.96 - 1.03 at 7168, 0.97 - 1.05
// beyond; W3A1 int32 0.99 - 1.02 at 8192, 1.02 - 1.05 at 9216; W4A1 0.86 - 0.99 throughout.
inline int64_t ksplit_lds_max_k(int p, int q, const GemmArgs &g)
{
    const bool i32_alone = !g.c_f16;
    if (p == 2) return !i32_alone ? 8704 : q == 3 ? 5632 : 7168;
    return p == 1 && q == 3 && i32_alone ? 8192 : 9216;
}
template <int P, int Q, int WM, int WN>
__global__ __launch_bounds__(WM == 4 ? 512 : 256, WN == 2 ? 2 : 1)  // two workgroups of the 64 x 64 tile share a compute unit
void gemm_mfma_ksplit_kernel(const uint32_t *a, const uint32_t *w, int32_t *c_i32, uint16_t *c_f16, int m, int n, int k, uint32_t magic, int tiles_n, int tiles_m_xn,
                             const uint16_t *w_scale, const uint16_t *a_scale, bool stream)
{
    extern __shared__ __align__(16) float4 red[];
    if constexpr (WM == 4) lds_tile<P, Q, 2, WN / 2, 2>(reinterpret_cast<uint4 *>(red), a, w, c_i32, c_f16, m, n, k, magic, tiles_n, tiles_m_xn, w_scale, a_scale, stream);
    else ksplit_tile<P, Q, WM, WN>(red, a, w, c_i32, c_f16, m, n, k, magic, tiles_n, tiles_m_xn, w_scale, a_scale, stream);
}
// The 128 x 256 tile (rule and figures: one_round_width): the same two groups of waves, each wave 64 x 128.  Start 3, k loop 17, exchange 1.4,
// store 2.6 us of W2A4 512 x 13824 x 5120; the products alone would take 10 in the loop, its LDS traffic 9.
template <int P, int Q>
__global__ __launch_bounds__(512, 1) void gemm_mfma_ksplit_wide_kernel(const uint32_t *a, const uint32_t *w, int32_t *c_i32, uint16_t *c_f16, int m, int n, int k,
                                                                       uint32_t magic, int tiles_n, int tiles_m_band, const uint16_t *w_scale,
                                                                       const uint16_t *a_scale, bool stream)
{
    extern __shared__ __align__(16) float4 red[];
    (void)c_i32;  // the rule takes an fp16 output alone: no code for the other
    lds_tile<P, Q, 2, 4, 2>(reinterpret_cast<uint4 *>(red), a, w, nullptr, c_f16, m, n, k, magic, tiles_n, tiles_m_band, w_scale, a_scale, stream);
}
template <int P, int Q>
__global__ __launch_bounds__(256) void gemm_mfma_ksplit_long_kernel(const uint32_t *a, const uint32_t *w, int32_t *c_i32, uint16_t *c_f16, int m, int n, int k,
                                                                    uint32_t magic, int tiles_n, int tiles_m_xn, const uint16_t *w_scale,
                                                                    const uint16_t *a_scale, bool stream)
{
    extern __shared__ __align__(16) float4 red[];
    ksplit_tile<P, Q, 4, 4>(red, a, w, c_i32, c_f16, m, n, k, magic, tiles_n, tiles_m_xn, w_scale, a_scale, stream);
}

template <int P, int Q, int WM, int WN>
hipError_t launch_ksplit_variant(const GemmArgs &g, hipStream_t stream)
{
    constexpr int BM = 32 * WM, BN = 32 * WN;
    const int64_t tiles_m = (g.M + BM - 1) / BM, tiles_n = (g.N + BN - 1) / BN;
    if (tiles_m >= (1 << 28) || tiles_n >= (1 << 28) || g.K > 0x7fffffffLL) return hipErrorInvalidValue;
    auto launch = [&](auto kernel, int64_t tiles, int threads, int lds, int order, uint32_t magic, bool streaming, int &prepared_device) {
        if (tiles > 0x7fffffffLL) return hipErrorInvalidValue;
        int dev = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return e;
        if (prepared_device != dev) {  // the LDS limit is a per-device attribute of the function
            e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
            if (e != hipSuccess) return e;
            prepared_device = dev;
        }
        const KernelTiming timing = take_kernel_timing();
        if (timing.start || timing.stop)
            hipExtLaunchKernelGGL(kernel, dim3((unsigned)tiles), dim3(threads), lds, stream, timing.start, timing.stop, 0, g.a, g.w,
                                  g.c_i32, g.c_f16, (int)g.M, (int)g.N, (int)g.K, magic, (int)tiles_n, order, g.w_scale, g.a_scale, streaming);
        else
            hipLaunchKernelGGL(kernel, dim3((unsigned)tiles), dim3(threads), lds, stream, g.a, g.w, g.c_i32, g.c_f16, (int)g.M, (int)g.N,
                               (int)g.K, magic, (int)tiles_n, order, g.w_scale, g.a_scale, streaming);
        return hipGetLastError();
    };
    static thread_local int prepared = -1, prepared_long = -1;
    if constexpr (WM == 4) {
        constexpr int lds = lds_tile_bytes<P, Q, 2, WN / 2, 2>();
        static_assert(lds <= 160 * 1024, "LDS of a compute unit");
        const int lds_order = lds_tile_order<P, Q>(tiles_m, g.K);
        if constexpr (WN == 8) {
            note_kernel("gemm_mfma_ksplit_wide_kernel<%d,%d>", P, Q);
            return launch(gemm_mfma_ksplit_wide_kernel<P, Q>, tiles_m * tiles_n, 512, lds, lds_order, lds_band_magic(lds_order, tiles_n, tiles_m * tiles_n),
                          lds_streams<P, Q, 2, WN / 2, 2>(g), prepared);
        } else if (Q == 2 || g.K <= ksplit_lds_max_k(P, Q, g)) {
            note_kernel("gemm_mfma_ksplit_kernel<%d,%d,%d,%d>", P, Q, WM, WN);
            return launch(gemm_mfma_ksplit_kernel<P, Q, WM, WN>, tiles_m * tiles_n, 512, lds, lds_order, lds_band_magic(lds_order, tiles_n, tiles_m * tiles_n),
                          lds_streams<P, Q, 2, WN / 2, 2>(g), prepared);
        }
    }
    // Parts of the tile grid per XCD: 8 / xn along M times xn along N, the cut that leaves an XCD the fewest packed
    // bytes to read (its row tiles of A plus its column tiles of W).
    int xn_log = 0;
    double best = 0;
    for (int l = 0; l <= 3; ++l) {
        const int64_t pm = (tiles_m + (8 >> l) - 1) / (8 >> l), pn = (tiles_n + (1 << l) - 1) / (1 << l);
        const double bytes = (double)pm * BM * activation_slots(P) + (double)pn * BN * Q;
        if (l == 0 || bytes < best) { best = bytes; xn_log = l; }
    }
    const int64_t part_m = (tiles_m + (8 >> xn_log) - 1) / (8 >> xn_log), part_n = (tiles_n + (1 << xn_log) - 1) / (1 << xn_log);
    const int order = (int)tiles_m | (xn_log << 28);
    const uint32_t magic = divisor_magic(part_m, part_m * part_n);
    if constexpr (WM != 4) {
        note_kernel("gemm_mfma_ksplit_kernel<%d,%d,%d,%d>", P, Q, WM, WN);
        return launch(gemm_mfma_ksplit_kernel<P, Q, WM, WN>, 8 * part_m * part_n, 256, ksplit_lds_bytes(WM, WN), order, magic, ksplit_streams(WM, WN, g), prepared);
    } else if constexpr (Q > 2 && WN == 4) {
        note_kernel("gemm_mfma_ksplit_long_kernel<%d,%d>", P, Q);
        return launch(gemm_mfma_ksplit_long_kernel<P, Q>, 8 * part_m * part_n, 256, ksplit_lds_bytes(WM, WN), order, magic, ksplit_streams(WM, WN, g), prepared_long);
    }
    return hipErrorInvalidValue;  // (not reached)
}

}  // namespace mfma
}  // namespace apmm
