// Design A for large outputs: the packed operands of a workgroup tile are shared through LDS.
//
// The algebra is that of apmm_gemm_mfma_direct.h (paper Sec. 3.2, the shift-and-add in front of the multiplier), and the operands are
// formed in registers from the packed words as there.  What differs is how the words come: there every wave loads all it needs for
// itself, one wave to a vector unit, and with 6-bit activation fields (and with the tiles that an output of several rounds gets)
// the k loop waits half of the time: two waves ask for every byte, a compute unit's L1 holds less than a stage of the tile, and
// in every second stage the compiler put the waits right behind the loads.  Here a byte comes to the compute unit once per tile,
// straight into LDS, and each wave reads its share from there, so that the registers hold little but accumulators and operands and
// two (AF: 6-bit fields) or three workgroups share a compute unit: while one meets at a barrier, starts, or stores its tile, the
// others multiply.  That is most of the gain: one workgroup to a compute unit, with all operands fetched a half stage ahead, takes
// 65.8 us for W2A4 4096 x 4096 x 8192, two 56.6, the direct kernel 77.4.  A ring of two half stages, which leaves LDS for three
// workgroups, is faster where there are many tiles of wide codes (W4A4 1024 x 11008 x 4096 0.65 against 0.69 of the direct time) and
// slower where there are few (512 x 13824 x 5120 0.98 against 0.85).
//
// Half stage = two k blocks, k steps 0, 1 or 2, 3 of each (lane l works on k block l / 32): the slots that those steps need, 16 KB of a
// 128 x 128 tile with 4-bit activations and 2-bit weights.  Four half stages are in LDS: the one in work, the next, whose first
// operands are formed under the end of this one, and two under way.  One barrier per half stage of 8 (128 x 128) or 16 (128 x 256) MFMAs.
// What bounds it: issue slots first, then LDS (128 x 256, W2A4: 60 KB read and written per 16 MFMAs of each vector unit, 117 B a clock at
// the full matrix rate, 80 reached); 22 - 24 ns per MFMA of 15 - 17.  Counters, W2A4 2048 x 11008 x 4096, W4A4 and W2A2 1024 x 11008 x 4096: matrix
// unit busy 60 / 43 / 55 %, a wave waits to issue for 38 / 31 / 40 % of its time, for data or a barrier 16 / 23 / 18 %, LDS reads active 21 / 30 / 17 %.
#pragma once
#include <hip/hip_ext.h>

#include <algorithm>

#include "apmm_mfma_common.h"

namespace apmm {
namespace mfma {

// A half stage is k steps 2 h, 2 h + 1 (h = 0, 1) of two k blocks.  Slots of a row that only one half uses, and slots that both
// use (they travel with the first half).
constexpr int lds_own_slots(int n, bool field) { return field ? 3 : n / 2; }
constexpr int lds_shared_slots(int n, bool field) { return !field && (n & 1) ? 1 : 0; }
constexpr int lds_own_slot(int n, bool field, int h, int i) { return field ? 3 * h + i : n == 4 ? 2 * h + i : h; }

constexpr int kLdsRing = 4;  // half stages in LDS
template <int P, int Q, int WM, int WN>
struct LdsTile {
    static constexpr bool AF = activation_field_form(P);
    static constexpr int RA = 2 * WM, RB = 2 * WN;  // row blocks of the workgroup tile
    static_assert(RA % 4 == 0 && RB % 4 == 0, "row blocks are dealt to four waves");
    static constexpr int OWN_A = lds_own_slots(P, AF), OWN_B = lds_own_slots(Q, false);
    static constexpr int SH_A = lds_shared_slots(P, AF), SH_B = lds_shared_slots(Q, false);
    static constexpr int HALF_VECS = 64 * (RA * OWN_A + RB * OWN_B), SHARED_VECS = 64 * (RA * SH_A + RB * SH_B);
    static constexpr int BYTES = 16 * (kLdsRing * HALF_VECS + kLdsRing / 2 * SHARED_VECS);
    // requests of one wave for a half stage
    static constexpr int loads(int h) { return RA / 4 * (OWN_A + (h == 0 ? SH_A : 0)) + RB / 4 * (OWN_B + (h == 0 ? SH_B : 0)); }
};

// 1 KB from memory to LDS: lane l's 16 bytes at base + voff + AT to lds + 16 l (the instruction's offset counts on both sides).  By
// hand: behind the builtin the compiler waits for every such load before any LDS read it cannot tell apart from it.  No register
// is written, so nothing can be reused early.
template <int AT>
__device__ __forceinline__ void load_to_lds(const char *base, uint32_t voff, uint32_t lds)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 offset:%3" ::"s"(lds - AT), "v"(voff), "s"(base), "n"(AT) : "memory", "m0");
}
// Everything this wave has read from LDS is in registers, all but its last N loads have arrived; then the same of every wave.
template <int N>
__device__ __forceinline__ void wait_and_meet()
{
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// Whether the workgroup that holds the first wave slots of a compute unit goes ahead of the others at every issue, so that it ends early and
// the tile of the second round runs under the others' k loop; those that run in step store together and leave that tile alone.  Each wave goes by
// its own slot: where waves of the kernel before still hold slots of some vector units, those of one workgroup differ and the gain is less
// (W2A4 2048 x 11008 x 4096 both, one behind the other 0.89 - 0.97, 61 - 65 -> 57 - 60 us, behind a packing 0.91 - 0.96, behind an elementwise kernel 0.95 - 0.98; one output
// 0.94 - 0.97 and 3-bit weights 0.91 - 0.98 in all three).
// Time with over without, operands and outputs in rotation:
// Two workgroups to a compute unit (3- and 4-bit activations), a round of 512 and up to 0.44 of a second.  128 x 256, 640 to 688 tiles, K = 2048 - 8192: both
// outputs 0.85 - 1.00, int32 0.91 - 1.00, fp16 0.94 - 1.01; K = 512 - 1536, where both are asked for, 0.97 - 1.05: not there.  864 and 960 tiles 0.99 - 1.02 and,
// both outputs, 1.06 - 1.18; 1376 1.02 - 1.05, 512 1.00 - 1.01.  128 x 128, 544 to 736 tiles: 3-bit weights 0.91 - 1.00 from K = 2048 on, 4-bit 0.95 - 1.01 from
// 2560 on (fp16 at 2048 up to 1.02); 1- and 2-bit 0.94 - 1.00 from 4096 on, at 2048 to 3072 0.96 - 1.03.
// Three workgroups (1- and 2-bit activations), 1.25 to 1.44 rounds of 768, in three steps, K = 2048 - 8192, 1032 to 1062 tiles: W2A2, W1A2 and W2A1 0.91 - 1.00 (946 tiles
// 0.98 - 1.01), with 4-bit weights 0.98 - 1.01; W1A1 0.97 - 1.06: not there.
template <int P, int Q, int WN>
__host__ __device__ constexpr bool lds_goes_ahead(int tiles, int k)
{
    if (activation_field_form(P)) return tiles > 512 && tiles <= 736 && k >= (WN == 4 || Q == 3 ? 2048 : Q == 4 ? 2560 : 4096);
    return Q <= 2 && P + Q > 2 && tiles > 960 && tiles <= 1104 && k >= 2048;
}

// One workgroup tile of 64 WM x 64 WN.  KG = 2: eight waves, the second four of which work on the second half of K with a ring of
// their own, for outputs of one round of tiles; in the end either group of waves adds up and stores one row block of each wave tile.
constexpr int lds_exchange_bytes(int wn) { return 8 * wn * 16 * 64 * 4; }
template <int P, int Q, int WM, int WN, int KG>
constexpr int lds_tile_bytes() { return KG == 1 ? LdsTile<P, Q, WM, WN>::BYTES : std::max(2 * LdsTile<P, Q, WM, WN>::BYTES, lds_exchange_bytes(WN)); }

template <int P, int Q, int WM, int WN, int KG>
__device__ __forceinline__ void lds_tile(uint4 *ring_of_workgroup, const uint32_t *a_arg, const uint32_t *w_arg, int32_t *ci_arg, uint16_t *cf_arg, int m_arg,
                                         int n_arg, int k_arg, uint32_t band_magic, int tiles_n, int tiles_m_band, const uint16_t *ws_arg,
                                         const uint16_t *as_arg, bool stream)
{
    using L = LdsTile<P, Q, WM, WN>;
    constexpr bool AF = L::AF;
    constexpr int SLOTS_A = activation_slots(P);
    constexpr int BM = 64 * WM, BN = 64 * WN;
    constexpr uint32_t ca = (1u << P) - 1, cw = (1u << Q) - 1;
    static_assert(KG == 1 || (KG == 2 && WM == 2), "the two groups of waves store a row block each");
    using I0 = std::integral_constant<int, 0>;

    const int lane = threadIdx.x & 63;
    const int wave_of_workgroup = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wave = KG == 1 ? wave_of_workgroup : wave_of_workgroup & 3, group = KG == 1 ? 0 : wave_of_workgroup >> 2;
    // [half stage % 4][row block][slot][lane], A before B; then the shared slots by stage % 2
    uint4 *ring = ring_of_workgroup + group * (L::BYTES / 16);
    const int wave_m = wave >> 1, wave_n = wave & 1;
    const int r32 = lane & 31, kh = lane >> 5;
    // An XCD takes a contiguous run of tiles in an order that walks `band` tile rows column by column (see lds_tile_order).
    // (All of the way to the first request is scalar arithmetic in 32 bits where the sizes allow it, 112 instead of 176 instructions for 128 x 256, with
    // which the median wave of a cold launch spent 1.0 us: W2A2 1024 x 11008 x 4096 int32 26.0 -> 25.7 us, W2A4 2048 x 11008 x 4096 both 62.3 -> 61.8.)
    const uint32_t nkb = padded_k_blocks(k_arg);
    const uint32_t tiles_m = tiles_m_band & 0x0fffffff, band_log = (uint32_t)tiles_m_band >> 28, band = 1u << band_log;
    const uint32_t lid = xcd_tile_id(blockIdx.x, tiles_n * (int)tiles_m);
    const uint32_t m_band = quotient(lid, (uint32_t)tiles_n << band_log, band_magic), in_band = lid - (m_band * tiles_n << band_log);
    const uint32_t rows = min(tiles_m - (m_band << band_log), band);  // 1, 2, 3 or 4
    const uint32_t tn = rows == 3 ? __umulhi(in_band, 0xaaaaaaabu) >> 1 : in_band >> (rows >> 1), tm = (m_band << band_log) + in_band - tn * rows;
    const int64_t M = m_arg, N = n_arg;
    const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;
    const uint32_t nrb_a = ((uint32_t)m_arg + 31) / 32, nrb_b = ((uint32_t)n_arg + 31) / 32;

    // What this wave brings to LDS: row blocks wave * RA / 4 ... of A and wave * RB / 4 ... of W (past the operand: the last one,
    // never stored).  Lane l takes row l % 32 of k block l / 32 of the stage, as it will read it.
    constexpr int kSlotBytes = kPlaneWords * 4;
    uint32_t voff_a = (uint32_t)(kh * SLOTS_A * kSlotBytes + r32 * 16);
    uint32_t voff_b = (uint32_t)(kh * Q * kSlotBytes + r32 * 16);
    const int stages = nkb / 2 / KG;  // this group's (nkb is a multiple of four)
    const char *src_a[L::RA / 4], *src_b[L::RB / 4];
#pragma unroll
    for (int i = 0; i < L::RA / 4; ++i) {
        const uint32_t rb = min(tm * (BM / 32) + wave * (L::RA / 4) + i, nrb_a - 1);
        src_a[i] = reinterpret_cast<const char *>(a_arg) + (uint64_t)(rb * nkb + group * 2 * stages) * (SLOTS_A * kSlotBytes);
    }
#pragma unroll
    for (int i = 0; i < L::RB / 4; ++i) {
        const uint32_t rb = min(tn * (BN / 32) + wave * (L::RB / 4) + i, nrb_b - 1);
        src_b[i] = reinterpret_cast<const char *>(w_arg) + (uint64_t)(rb * nkb + group * 2 * stages) * (Q * kSlotBytes);
    }
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint4 *)ring;
    // Requests go half stage by half stage; this one is for ring place `r` (its parity is the half).  Past the last stage every lane
    // asks for the same 16 bytes, so that the number of requests under way stays what the waits count on.
    int to_request = stages;
    auto request_one = [&](auto r_c, auto n_c) __attribute__((always_inline)) {
        constexpr int r = decltype(r_c)::value, h = r & 1, n = decltype(n_c)::value;
        constexpr int per_a = L::OWN_A + (h == 0 ? L::SH_A : 0), per_b = L::OWN_B + (h == 0 ? L::SH_B : 0), all_a = L::RA / 4 * per_a;
        constexpr uint32_t kShared = kLdsRing * L::HALF_VECS + r / 2 * L::SHARED_VECS;
        if constexpr (n < all_a) {
            constexpr int i = n / per_a, s = n % per_a;
            const int blk = wave * (L::RA / 4) + i;
            if constexpr (s < L::OWN_A)
                load_to_lds<lds_own_slot(P, AF, h, s) * kSlotBytes>(src_a[i], voff_a, lds0 + 16 * (r * L::HALF_VECS + 64 * (blk * L::OWN_A + s)));
            else load_to_lds<(P - 1) * kSlotBytes>(src_a[i], voff_a, lds0 + 16 * (kShared + 64 * blk));
        } else {
            constexpr int i = (n - all_a) / per_b, s = (n - all_a) % per_b;
            const int blk = wave * (L::RB / 4) + i;
            if constexpr (s < L::OWN_B)
                load_to_lds<lds_own_slot(Q, false, h, s) * kSlotBytes>(src_b[i], voff_b,
                                                                       lds0 + 16 * (r * L::HALF_VECS + 64 * (L::RA * L::OWN_A + blk * L::OWN_B + s)));
            else load_to_lds<(Q - 1) * kSlotBytes>(src_b[i], voff_b, lds0 + 16 * (kShared + 64 * (L::RA * L::SH_A + blk)));
        }
    };
    auto next_stage = [&]() __attribute__((always_inline)) {
        --to_request;
        const int step = to_request > 0 ? 1 : 0;
        if (to_request <= 0) voff_a = voff_b = 0;
#pragma unroll
        for (int i = 0; i < L::RA / 4; ++i) src_a[i] += step * 2 * SLOTS_A * kSlotBytes;
#pragma unroll
        for (int i = 0; i < L::RB / 4; ++i) src_b[i] += step * 2 * Q * kSlotBytes;
    };
    auto request = [&](auto r_c) __attribute__((always_inline)) {
        constexpr int h = decltype(r_c)::value & 1;
        static_for<L::loads(h)>([&](auto n_c) __attribute__((always_inline)) { request_one(r_c, n_c); });
        if constexpr (h == 1) next_stage();
    };
    static_for<kLdsRing - 1>(request);
    if constexpr (KG == 1) {
        if (lds_goes_ahead<P, Q, WN>(tiles_n * (int)tiles_m, k_arg)) {
            constexpr int kHwId = 4, kSlotBits = 4;  // the register that says where a wave runs; its lowest field is the slot in the vector unit
            const uint32_t slot = __builtin_amdgcn_s_getreg(kHwId | (kSlotBits - 1) << 11);
            if constexpr (AF) {
                if ((slot & 1) == 0) __builtin_amdgcn_s_setprio(1);
            } else {
                if (slot == 0) __builtin_amdgcn_s_setprio(2);
                else if (slot == 1) __builtin_amdgcn_s_setprio(1);
            }
        }
    }

    // For the end of the tile, requested now: code sums and scales of this lane's columns and rows.
    const int32_t *a_sum = reinterpret_cast<const int32_t *>(a_arg) + (uint64_t)(nrb_a * nkb) * (kRowBlock * SLOTS_A * 4);
    const int32_t *w_sum = reinterpret_cast<const int32_t *>(w_arg) + (uint64_t)(nrb_b * nkb) * (kRowBlock * Q * 4);
    constexpr int WMO = WM / KG;  // row blocks of the wave tile that this wave finishes, the first of them:
    const int64_t m_own = m0 + (wave_m * WM + group) * 32, m_lane = m_own + kh * 4, n_lane = n0 + wave_n * WN * 32 + r32;
    uint32_t w_sum_raw[WN], a_sum_raw[WMO], sw_raw[WN], sa_raw[(WMO + 1) / 2];
#pragma unroll
    for (int bj = 0; bj < WN; ++bj) {
        w_sum_raw[bj] = (uint32_t)w_sum[min((uint32_t)n_lane + bj * 32, nrb_b * 32 - 1)];
        sw_raw[bj] = 0x3c00u;  // 1.0
    }
#pragma unroll
    for (int bi = 0; bi < WMO; ++bi) {
        a_sum_raw[bi] = (uint32_t)a_sum[min((uint32_t)m_own + bi * 32 + r32, nrb_a * 32 - 1)];
    }
#pragma unroll
    for (int i = 0; i < (WMO + 1) / 2; ++i) sa_raw[i] = 0x3c00u;
    if (cf_arg && ws_arg) {
#pragma unroll
        for (int bj = 0; bj < WN; ++bj) {
            sw_raw[bj] = ws_arg[min((uint32_t)n_lane + bj * 32, (uint32_t)n_arg - 1)];
        }
    }
    if (cf_arg && as_arg) {
#pragma unroll
        for (int i = 0; i < (WMO + 1) / 2; ++i) {
            sa_raw[i] = as_arg[min((uint32_t)m_own + 64 * i + lane, (uint32_t)m_arg - 1)];
        }
    }

    v16f acc[WM][WN];
#pragma unroll
    for (int bi = 0; bi < WM; ++bi)
#pragma unroll
        for (int bj = 0; bj < WN; ++bj)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[bi][bj][v] = 0.f;

    // Raw words of a half stage and of a stage (shared slots), formed operands by k step parity.
    uint4 ra[WM][L::OWN_A ? L::OWN_A : 1], rb[WN][L::OWN_B ? L::OWN_B : 1], ra_sh[L::SH_A ? WM : 1], rb_sh[L::SH_B ? WN : 1];
    v4i af[2][AF ? 1 : WM];
    uint2 am[2][AF ? WM : 1];
    OperandFrag<Q> bf[2][WN];
    const uint4 *mine_a = ring + wave_m * WM * L::OWN_A * 64 + lane, *mine_b = ring + (L::RA * L::OWN_A + wave_n * WN * L::OWN_B) * 64 + lane;
    const uint4 *mine_sa = ring + kLdsRing * L::HALF_VECS + wave_m * WM * 64 + lane;
    const uint4 *mine_sb = ring + kLdsRing * L::HALF_VECS + (L::RA * L::SH_A + wave_n * WN) * 64 + lane;
    // The reads of a half stage in the order of their first uses; the last of a field operand's three slots is used by the second k
    // step alone and comes at the end.
    constexpr int kFetches[2] = {WM * (L::OWN_A + L::SH_A) + WN * (L::OWN_B + L::SH_B), WM * L::OWN_A + WN * L::OWN_B};  // by half
    auto fetch = [&](auto r_c, auto n_c) __attribute__((always_inline)) {
        constexpr int r = decltype(r_c)::value, h = r & 1, n = decltype(n_c)::value;
        constexpr int sh_a = h == 0 ? L::SH_A : 0, sh_b = h == 0 ? L::SH_B : 0;
        constexpr int mid = AF ? WM : 0, b0 = mid + (L::OWN_B ? WN : 0), sb = b0 + sh_b * WN, sa = sb + sh_a * WM, a0 = sa + (L::OWN_A ? WM : 0),
                      b1 = a0 + (L::OWN_B > 1 ? WN : 0);
        if constexpr (n < mid) ra[n][1] = mine_a[r * L::HALF_VECS + (n * L::OWN_A + 1) * 64];
        else if constexpr (n < b0) rb[n - mid][0] = mine_b[r * L::HALF_VECS + (n - mid) * L::OWN_B * 64];
        else if constexpr (n < sb) rb_sh[n - b0] = mine_sb[r / 2 * L::SHARED_VECS + (n - b0) * 64];
        else if constexpr (n < sa) ra_sh[n - sb] = mine_sa[r / 2 * L::SHARED_VECS + (n - sb) * 64];
        else if constexpr (n < a0) ra[n - sa][0] = mine_a[r * L::HALF_VECS + (n - sa) * L::OWN_A * 64];
        else if constexpr (n < b1) rb[n - a0][1] = mine_b[r * L::HALF_VECS + ((n - a0) * L::OWN_B + 1) * 64];
        else ra[n - b1][2] = mine_a[r * L::HALF_VECS + ((n - b1) * L::OWN_A + 2) * 64];
    };
    auto fetch_range = [&](auto r_c, auto from_c, auto to_c) __attribute__((always_inline)) {
        constexpr int from = decltype(from_c)::value, to = decltype(to_c)::value;
        static_for<(to > from ? to - from : 0)>([&](auto n_c) __attribute__((always_inline)) {
            fetch(r_c, std::integral_constant<int, from + decltype(n_c)::value>{});
        });
    };
    constexpr int TASKS_A = (AF ? 2 : 4) * WM, DB = operand_dwords(Q), TASKS = TASKS_A + DB * WN, PER_KS = WM * WN;
    // operand dword `task` of local k step ksl of the half stage at ring place r
    auto form = [&](auto r_c, auto ksl_c, auto task_c) __attribute__((always_inline)) {
        constexpr int r = decltype(r_c)::value, h = r & 1, ksl = decltype(ksl_c)::value, task = decltype(task_c)::value;
        if constexpr (task < TASKS_A) {
            constexpr int f = task / (AF ? 2 : 4), d = task % (AF ? 2 : 4);
            if constexpr (AF) {
                if constexpr (d == 0) am[ksl][f].x = copy_here(vec_word<2 * ksl>(ra[f][1]));
                else am[ksl][f].y = copy_here(vec_word<2 * ksl + 1>(ra[f][1]));
            } else {
                uint4 raw[1];
                if constexpr (P == 1) raw[0] = ra_sh[f];
                else raw[0] = ra[f][0];
                af[ksl][f][d] = (int)half_operand_dword<P, h, ksl, d>(raw);
            }
        } else {
            constexpr int f = (task - TASKS_A) / DB, d = (task - TASKS_A) % DB;
            uint4 raw[half_slots(Q, false)];
            if constexpr (Q == 1) raw[0] = rb_sh[f];
            else raw[0] = rb[f][0];
            if constexpr (Q == 3) raw[1] = rb_sh[f];
            if constexpr (Q == 4) raw[1] = rb[f][1];
            bf[ksl][f][d] = (int)half_operand_dword<Q, h, ksl, d>(raw);
        }
    };
    // One half stage, its first operands formed and its raw words in registers, but for the last slot of field operands.
    auto half = [&](auto r_c) __attribute__((always_inline)) {
        constexpr int r = decltype(r_c)::value, h = r & 1;
        static_assert(L::loads(h ^ 1) < 2 * PER_KS, "a request per MFMA");
        using Next = std::integral_constant<int, (r + 1) % kLdsRing>;
        using Request = std::integral_constant<int, (r + kLdsRing - 1) % kLdsRing>;
        // the half stage after this one has to be there now, this wave's requests for the one behind it may be under way
        wait_and_meet<L::loads(h)>();
        __builtin_amdgcn_sched_barrier(0);
        static_for<2 * PER_KS>([&](auto i_c) __attribute__((always_inline)) {
            constexpr int i = decltype(i_c)::value, ksl = i / PER_KS, j = i % PER_KS, bi = j / WN, bj = j % WN;
            constexpr int TPM = (TASKS + PER_KS - 1 - 1) / (PER_KS - 1);  // tasks per MFMA; none under the first of a k step
            constexpr int format_a = operand_format(P), format_b = operand_format(Q);
            if constexpr (j == 0) {
                constexpr int late = AF ? WM : 0;
                if constexpr (ksl == 0) fetch_range(r_c, std::integral_constant<int, kFetches[h] - late>{}, std::integral_constant<int, kFetches[h]>{});
                else fetch_range(Next{}, I0{}, std::integral_constant<int, kFetches[h ^ 1] - late>{});
                __builtin_amdgcn_sched_barrier(0);
            }
            v8i a8;
            if constexpr (AF) a8 = field_operand<ksl>(ra[bi], am[ksl][bi]);
            else a8 = widen(af[ksl][bi]);
            acc[bi][bj] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a8, widen(bf[ksl][bj]), acc[bi][bj], format_a, format_b, 0,
                                                                        operand_exponent(P, 2 * h + ksl), 0, operand_exponent(Q, 2 * h + ksl));
            if constexpr (i < L::loads(h ^ 1)) request_one(Request{}, i_c);
            if constexpr (h == 0 && i == L::loads(1)) next_stage();
            if constexpr (j > 0) {
                static_for<TPM>([&](auto t_c) __attribute__((always_inline)) {
                    constexpr int task = (j - 1) * TPM + decltype(t_c)::value;
                    if constexpr (task < TASKS) {
                        using X = std::integral_constant<int, task>;
                        if constexpr (ksl == 0) form(r_c, std::integral_constant<int, 1>{}, X{});
                        else form(Next{}, I0{}, X{});
                    }
                });
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    wait_and_meet<L::loads(1) + L::loads(0)>();
    fetch_range(I0{}, I0{}, std::integral_constant<int, kFetches[0]>{});
    static_for<TASKS>([&](auto t_c) __attribute__((always_inline)) { form(I0{}, I0{}, t_c); });
    int st = 0;
    for (; st + 1 < stages; st += kLdsRing / 2) static_for<kLdsRing>(half);
    if constexpr (KG == 2) {
        if (st < stages) static_for<kLdsRing / 2>(half);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // nothing may still be on its way to LDS when the workgroup ends

    v16f c[WMO][WN];
    if constexpr (KG == 1) {
#pragma unroll
        for (int bi = 0; bi < WM; ++bi)
#pragma unroll
            for (int bj = 0; bj < WN; ++bj) c[bi][bj] = acc[bi][bj];
    } else {
        // Either group hands the other one's row block over (fp32 sums of integers below 2^24: exact in any order).
        float4 *there = reinterpret_cast<float4 *>(ring_of_workgroup) + (wave_of_workgroup ^ 4) * WN * 256 + lane;
        const float4 *here = reinterpret_cast<const float4 *>(ring_of_workgroup) + wave_of_workgroup * WN * 256 + lane;
        __syncthreads();  // the rings are read
#pragma unroll
        for (int bj = 0; bj < WN; ++bj)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float4 give;
                give.x = group ? acc[0][bj][4 * i] : acc[1][bj][4 * i];
                give.y = group ? acc[0][bj][4 * i + 1] : acc[1][bj][4 * i + 1];
                give.z = group ? acc[0][bj][4 * i + 2] : acc[1][bj][4 * i + 2];
                give.w = group ? acc[0][bj][4 * i + 3] : acc[1][bj][4 * i + 3];
                there[(bj * 4 + i) * 64] = give;
            }
        __syncthreads();
#pragma unroll
        for (int bj = 0; bj < WN; ++bj)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float4 got = here[(bj * 4 + i) * 64];
                c[0][bj][4 * i] = (group ? acc[1][bj][4 * i] : acc[0][bj][4 * i]) + got.x;
                c[0][bj][4 * i + 1] = (group ? acc[1][bj][4 * i + 1] : acc[0][bj][4 * i + 1]) + got.y;
                c[0][bj][4 * i + 2] = (group ? acc[1][bj][4 * i + 2] : acc[0][bj][4 * i + 2]) + got.z;
                c[0][bj][4 * i + 3] = (group ? acc[1][bj][4 * i + 3] : acc[0][bj][4 * i + 3]) + got.w;
            }
    }

    // The recovery terms rt[m] + ct[n], rt = -2 cw PA, ct = K ca cw - 2 ca PW: one fp32 MFMA with k = 2 per block, A = (rt[m], 1),
    // B = (1, ct[n]); lane l supplies row resp. column l % 32 of k index l / 32.
    float b_fin[WN], a_fin[WMO], sw[WN];
#pragma unroll
    for (int bj = 0; bj < WN; ++bj) {
        const float ct = (float)(int32_t)((uint32_t)k_arg * ca * cw - 2u * ca * use_here(w_sum_raw[bj]));
        b_fin[bj] = kh == 0 ? 1.0f : ct;
        sw[bj] = half_bits_to_float((uint16_t)use_here(sw_raw[bj]));
    }
#pragma unroll
    for (int bi = 0; bi < WMO; ++bi) {
        const float rt = -(float)(2u * cw * use_here(a_sum_raw[bi]));
        a_fin[bi] = kh == 0 ? rt : 1.0f;
    }
#pragma unroll
    for (int bi = 0; bi < WMO; ++bi)
#pragma unroll
        for (int bj = 0; bj < WN; ++bj) c[bi][bj] = __builtin_amdgcn_mfma_f32_32x32x2f32(a_fin[bi], b_fin[bj], c[bi][bj], 0, 0, 0);

    // Store, as in apmm_gemm_mfma_direct.h: one pass per output, fp16 in pairs of columns where the addresses allow it, streaming stores by
    // the rule of lds_streams (but single fp16 elements behind an int32 output, odd widths: plain, 1500 x 5003 x 3001 W2A4 28.8 against
    // 23.3 us).  Streaming fp16 pairs: all words of two rows, then their stores, so that the pieces of a line, 64 bytes of each row, leave one right behind the
    // other; apart by the operations for a piece the memory system joins fewer of them.  That needs the token scales of a block at hand, their lane permutes
    // requested together, or a workgroup that is alone waits for each.  2048 x 4096 fp16, piece by piece with twelve operations a pair / with six / together:
    // W2A4 K = 512 8.2 / 9.0 / 7.6 us, K = 1024 10.0 / 10.7 / 9.2, W4A4 K = 512 10.4 / 10.5 / 9.6; 2048 x 12288 x 512 W1A1 17.0 / 18.6 / 15.3, W2A4 20.5 / 21.9 / 19.9; 512 x 4096 x 512
    // W4A4 5.7 / 5.7 / 5.7, without the scales at hand 5.9.  (Plain stores meet in L2 in any order: both outputs 1.00 - 1.02 with it.)
    auto emit = [&](auto guard_c, auto i32_c, auto f16_c, auto pair_c, auto nt_c) __attribute__((always_inline)) {
        constexpr bool GUARD = decltype(guard_c)::value, I32 = decltype(i32_c)::value, F16 = decltype(f16_c)::value,
                       PAIR = decltype(pair_c)::value, NT = decltype(nt_c)::value;
        constexpr bool TOGETHER = F16 && PAIR && NT;  // the 64-byte pieces of a line leave one right behind the other
        if constexpr (NT) edge_of_streaming();
        int32_t *ci = I32 ? ci_arg + m_lane * N + n_lane : nullptr;
        uint16_t *ch = F16 ? cf_arg + m_lane * N + n_lane : nullptr;
        const bool odd = lane & 1;
        uint16_t *ch_pair = F16 ? ch + (odd ? N - 1 : 0) : nullptr;  // odd lanes write the row below at the column to the left
        const uint32_t selector = swap_pair_selector(odd);
        auto token_scale = [&](int bi, int v) __attribute__((always_inline)) {
            const uint32_t h = (uint32_t)__shfl((int)sa_raw[bi / 2], (bi & 1) * 32 + 8 * (v / 4) + 4 * kh + (v % 4));
            return half_bits_to_float((uint16_t)h);
        };
#pragma unroll
        for (int bi = 0; bi < WMO; ++bi) {
            float sa_of[16];
            if constexpr (TOGETHER) {  // (one wait for all of them)
#pragma unroll
                for (int v = 0; v < 16; ++v) sa_of[v] = token_scale(bi, v);
#pragma unroll
                for (int v = 0; v < 16; ++v) asm volatile("" : "+v"(sa_of[v]));
            }
            auto scale_of = [&](int v) __attribute__((always_inline)) { return TOGETHER ? sa_of[v & 15] : token_scale(bi, v); };
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int64_t row = (int64_t)(bi * 32 + 8 * (v / 4) + (v % 4));
                // the lane permutes come before any lane leaves the iteration: a lane that has left supplies nothing
                const float sa = F16 ? scale_of(v) : 1.0f;
                const float sa_next = (F16 && PAIR && v % 2 == 0) ? scale_of(v + 1) : 1.0f;
                if (GUARD && m_lane + row >= M) continue;
#pragma unroll
                for (int bj = 0; bj < WN; ++bj) {
                    if (GUARD && n_lane + bj * 32 >= N) continue;
                    const float x = c[bi][bj][v];
                    if constexpr (I32 && NT) __builtin_nontemporal_store((int32_t)x, &ci[row * N + bj * 32]);
                    if constexpr (I32 && !NT) ci[row * N + bj * 32] = (int32_t)x;
                    if constexpr (F16 && !PAIR) {
                        if constexpr (NT) __builtin_nontemporal_store(float_to_half_bits(x * sa * sw[bj]), &ch[row * N + bj * 32]);
                        else ch[row * N + bj * 32] = float_to_half_bits(x * sa * sw[bj]);
                    }
                }
                if constexpr (F16 && PAIR) {
                    if (v % 2 == 0) {
                        uint32_t word[WN];
#pragma unroll
                        for (int bj = 0; bj < WN; ++bj) word[bj] = swap_pair(half_pair(c[bi][bj][v] * sa, c[bi][bj][(v + 1) & 15] * sa_next, sw[bj]), selector);
#pragma unroll
                        for (int bj = 0; bj < WN; ++bj)
                            if constexpr (TOGETHER) asm volatile("" : "+v"(word[bj]));
#pragma unroll
                        for (int bj = 0; bj < WN; ++bj) {
                            uint32_t *dst = reinterpret_cast<uint32_t *>(ch_pair + row * N + bj * 32);
                            if constexpr (NT) __builtin_nontemporal_store(word[bj], dst);
                            else *dst = word[bj];
                        }
                    }
                }
            }
        }
        if constexpr (NT) edge_of_streaming();
    };
    using T = std::true_type;
    using F = std::false_type;
    const bool interior = (m0 + BM <= M) && (n0 + BN <= N);
    const bool pair = (N & 1) == 0 && (reinterpret_cast<uintptr_t>(cf_arg) & 3u) == 0;
    if (ci_arg) {
        if (interior && stream) emit(F{}, T{}, F{}, F{}, T{});
        else if (interior) emit(F{}, T{}, F{}, F{}, F{});
        else emit(T{}, T{}, F{}, F{}, F{});
    }
    if (cf_arg) {
        if (interior && pair && stream) emit(F{}, F{}, T{}, T{}, T{});
        else if (interior && pair) emit(F{}, F{}, T{}, T{}, F{});
        else if (interior && stream && !ci_arg) emit(F{}, F{}, T{}, F{}, T{});
        else if (interior) emit(F{}, F{}, T{}, F{}, F{});
        else emit(T{}, F{}, T{}, F{}, F{});
    }
}

template <int P, int Q, int WM, int WN, int OCC>
__global__ __launch_bounds__(256, OCC) void gemm_mfma_lds_kernel(const uint32_t *a, const uint32_t *w, int32_t *c_i32, uint16_t *c_f16, int m, int n, int k,
                                                                 uint32_t band_magic, int tiles_n, int tiles_m_band, const uint16_t *w_scale,
                                                                 const uint16_t *a_scale, bool stream)
{
    extern __shared__ __align__(16) uint4 lds_ring[];
    lds_tile<P, Q, WM, WN, 1>(lds_ring, a, w, c_i32, c_f16, m, n, k, band_magic, tiles_n, tiles_m_band, w_scale, a_scale, stream);
}

template <int P, int Q>
inline int lds_tile_order(int64_t tiles_m, int64_t K)  // tiles_m < 2^28
{
    // Order of the tiles.  Four tile rows walked column by column let the workgroups that run together on an XCD share the packed rows
    // of four tile rows and of the columns under way in its L2; row by row, they write longer runs of C.  The latter pays where the
    // operands are light.  Microseconds, row by row / in fours, both outputs: 4096 x 11008 x 1024 W2A4 65 / 71, W2A2 65 / 69, W1A2 64 /
    // 69, W4A4 76 / 69; 3000 x 8000 x 700 W2A4 40 / 39, W4A4 44 / 40; 2048 x 11008 x 4096 W2A2 57 / 53, W4A4 79 / 71.  (In eights: W2A4 4096 x
    // 11008 x 1024 78, 2048 x 11008 x 4096 W2A4 63 against 60.)
    const int band_log = Q <= 2 && K <= 1024 ? 0 : 2;
    return (int)tiles_m | band_log << 28;
}
inline uint32_t lds_band_magic(int tiles_m_band, int64_t tiles_n, int64_t tiles) { return divisor_magic(tiles_n << (tiles_m_band >> 28), tiles); }

// Streaming stores where the rows are whole lines: with outputs that are not in the last-level cache from the call before, plain ones
// push the operands out of L2 (W2A4 1024 x 11008 x 4096 both 33.6 -> 43.4 us, int32 28.8 -> 37.0, fp16 28.0 -> 35.7).  Not where a short sum
// leaves both outputs to be all there is to do, K up to 512 or up to 2.4e10 products, from 45 MB on (128 x 128 with fields: up to 80 MB): plain
// over streaming at 60 - 80 MB 0.84 / 0.86 / 0.91 / 0.98 with K = 512 / 1024 / 2048 / 3072 (1- and 2-bit activations; 3 and 4 bits 0.91 - 0.96), at 80 -
// 120 MB 0.89 / 0.96 / 1.03 / 1.06 (0.97 / 1.06 / 1.08 / 1.09), at 200 MB 0.86 / 0.99 / 1.20 (1.08 / 1.24 / 1.34).  int32 alone under 1- and 2-bit
// activations, K up to 512: 0.80 - 1.02 at 45 - 90 MB (1500 x 8000 1.05), 1.05 - 1.12 at 134.  Rows of parts of lines: also where the
// operands of a tile row and column, K slots wide, fill an L2 and lose more to plain stores (W4A4 1024 x 11016 with K = 4096 / 6144 / 8192 /
// 11008 both plain over streaming 1.02 / 1.17 / 1.18 / 1.13, W2A4 0.85 / 0.95 / 1.10 / 1.20).
template <int P, int Q, int WM, int WN, int KG>
inline bool lds_streams(const GemmArgs &g)
{
    const OutputRows rows(g);
    if (KG == 2 && !rows.both) return true;
    if (!rows.whole) return rows.fit_l2() || g.K * (activation_slots(P) + Q) >= 60000;
    const bool few = g.M * g.N * g.K <= 24000000000;
    const bool short_sum = activation_field_form(P) && WN == 2 ? few && rows.bytes < 80000000 : few || g.K <= 512;
    if (!rows.both) return !(P <= 2 && g.c_i32 && g.K <= 512 && rows.bytes >= 44000000 && rows.bytes < 100000000);
    return rows.bytes < 45000000 || !short_sum;
}

template <int P, int Q, int WM, int WN, int OCC>
hipError_t launch_lds_variant(const GemmArgs &g, hipStream_t stream)
{
    using L = LdsTile<P, Q, WM, WN>;
    static_assert(L::BYTES * OCC <= 160 * 1024, "the rings of the workgroups of a compute unit must fit its LDS");
    const int64_t tiles_m = (g.M + 64 * WM - 1) / (64 * WM), tiles_n = (g.N + 64 * WN - 1) / (64 * WN);
    const int64_t tiles = tiles_m * tiles_n;
    if (tiles > 0x7fffffffLL || tiles_m >= (1 << 28) || g.M > 0x7fffffffLL || g.N > 0x7fffffffLL || g.K > 0x7fffffffLL) return hipErrorInvalidValue;
    const int tiles_m_band = lds_tile_order<P, Q>(tiles_m, g.K);
    const uint32_t magic = lds_band_magic(tiles_m_band, tiles_n, tiles);
    const bool streaming = lds_streams<P, Q, WM, WN, 1>(g);
    auto kernel = gemm_mfma_lds_kernel<P, Q, WM, WN, OCC>;
    static thread_local int prepared_device = -1;  // the LDS limit is a per-device attribute of the function
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (prepared_device != dev) {
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, L::BYTES);
        if (e != hipSuccess) return e;
        prepared_device = dev;
    }
    const KernelTiming timing = take_kernel_timing();
    note_kernel("gemm_mfma_lds_kernel<%d,%d,%d,%d>", P, Q, WM, WN);
    if (timing.start || timing.stop)
        hipExtLaunchKernelGGL(kernel, dim3((unsigned)tiles), dim3(256), L::BYTES, stream, timing.start, timing.stop, 0, g.a, g.w, g.c_i32,
                              g.c_f16, (int)g.M, (int)g.N, (int)g.K, magic, (int)tiles_n, tiles_m_band, g.w_scale, g.a_scale, streaming);
    else
        hipLaunchKernelGGL(kernel, dim3((unsigned)tiles), dim3(256), L::BYTES, stream, g.a, g.w, g.c_i32, g.c_f16, (int)g.M, (int)g.N,
                           (int)g.K, magic, (int)tiles_n, tiles_m_band, g.w_scale, g.a_scale, streaming);
    return hipGetLastError();
}

}  // namespace mfma
}  // namespace apmm
