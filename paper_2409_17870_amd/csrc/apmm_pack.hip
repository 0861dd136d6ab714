// Pack / unpack kernels: paper Sec. 4.1 (matrix decomposition and reassembly).
//   step 1  split every code into its bits (planes)
//   step 2  reassemble the planes into 32-bit words
//   step 3  concatenate them (here: tile-interleaved and grouped for the consumers, see apmm_layout.h)
// plus, behind the tiles, one int32 per row: the sum of the row's codes over the padded K, which the
// MFMA kernels need for the recovery and which costs one byte-sum per four codes here instead of
// popcounts per word and output tile there.
//
// Widths and row ends are compile-time (a launch fetches only the code it runs: one 4096-code row of two bits 2.4 ->
// 2.2 us, 64 rows 2.6 -> 2.3 us).
//
// pack_kernel works tile by tile (one wave per 32 rows x 128 k, whole cache lines written by one instruction)
// with separate waves for the code sums, pack_eights_kernel by eight rows with the sums on the way (many rows); pack_rows_kernel and the fused quantise + pack kernel work row by row
// (one wave or a few per row; the quantiser has to see the whole row for its scale first).  No atomics.  The work is HBM bound: 1 byte
// read and bits/8 bytes written per element.
#include <hip/hip_fp16.h>

#include <type_traits>

#include "apmm_kernels.h"

namespace apmm {
namespace {

constexpr int kThreads = 256;
constexpr int kRowsPerWg = kThreads / 64;

// The wave's number as a scalar, and with it everything that follows from it: rows, bases, the branches between kinds of waves.
__device__ __forceinline__ int wave_of_workgroup() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }

// Sum and maximum over the 64 lanes, as a scalar: lane permutes inside the vector unit, six instructions where shuffles through LDS
// are six round trips (1 x 4096 two bits 2.27 -> 2.19 us, quantised to four 3.1 -> 2.85).  0 is neutral for both.
template <class Op>
__device__ __forceinline__ uint32_t over_wave(uint32_t v, Op op)
{
    v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false));  // row_shr 1, 2, 4, 8: lane 15 of 16 has its row's
    v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false));
    v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false));
    v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false));
    v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false));  // row_bcast 15 into rows 1 and 3
    v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false));  // row_bcast 31 into rows 2 and 3
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}
__device__ __forceinline__ uint32_t sum_over_wave(uint32_t v)
{
    return over_wave(v, [](uint32_t a, uint32_t b) __attribute__((always_inline)) { return a + b; });
}
__device__ __forceinline__ uint32_t max_over_wave(uint32_t v)
{
    return over_wave(v, [](uint32_t a, uint32_t b) __attribute__((always_inline)) { return a > b ? a : b; });
}

// nibbles of the four codes in lo (jh = 0) and in hi (jh = 1)
__device__ __forceinline__ uint32_t nibble_word(uint32_t lo, uint32_t hi)
{
    return (lo & 0x0f0f0f0fu) | ((hi & 0x0f0f0f0fu) << 4);
}

// 4 * NW codes of a row from k0 on, at any alignment (unaligned 16-byte and dword loads are single instructions here).
// WHOLE: K is a multiple of 4 NW, a piece lies inside the row or past it.  Else a piece that crosses the row's end takes dwords clamped to the last four codes and shifts the ones that lie before it
// out; positions past K become 0xff (pad: every plane bit set).  All loads of a piece are in flight together: byte loads
// under a condition each, the earlier form, waited one by one (fresh 5003 x 3001 and 1000 x 3001 three-bit codes, packing
// and product: 103 -> 47 us).
struct __attribute__((packed, aligned(1))) AnyVec { uint32_t x, y, z, w; };
struct __attribute__((packed, aligned(1))) AnyWord { uint32_t x; };
struct __attribute__((packed, aligned(4))) WordVec { uint32_t x, y, z, w; };

// The 4 NW bytes from `src` on, at any alignment, out of whole dwords: a 16-byte load that does not start at a dword takes several
// times as long (5003 x 3001 three-bit codes 9.6 -> 7.1 us; 5003 x 3008 5.9).  Every dword read holds one of the bytes.
template <int NW>
__device__ __forceinline__ void load_bytes(const void *src, uint32_t (&d)[NW])
{
    const uint32_t shift = (uint32_t)reinterpret_cast<uintptr_t>(src) & 3u;
    const uint32_t *words = reinterpret_cast<const uint32_t *>(reinterpret_cast<uintptr_t>(src) - shift);
    uint32_t w[NW + 1];
#pragma unroll
    for (int i = 0; i < NW / 4; ++i) {
        const WordVec v = reinterpret_cast<const WordVec *>(words)[i];
        w[4 * i] = v.x; w[4 * i + 1] = v.y; w[4 * i + 2] = v.z; w[4 * i + 3] = v.w;
    }
    w[NW] = words[shift ? NW : NW - 1];
#pragma unroll
    for (int i = 0; i < NW; ++i) d[i] = __builtin_amdgcn_alignbyte(w[i + 1], w[i], shift);
}

template <bool WHOLE, int NW>
__device__ __forceinline__ void load_codes(const uint8_t *__restrict__ row, int64_t K, int64_t k0, uint32_t (&d)[NW])
{
    const uint8_t *src = row + k0;
    // (eight dwords in a row of a wave's own are not faster that way: 200 x 5001 two-bit codes 3.3 -> 3.5 us)
    if (!WHOLE && NW > 8 && k0 + 4 * NW <= K && ((K | (int64_t)reinterpret_cast<uintptr_t>(row)) & 3) != 0) {
        load_bytes<NW>(src, d);
    } else if (k0 + 4 * NW <= K) {
#pragma unroll
        for (int i = 0; i < NW / 4; ++i) {
            const AnyVec v = reinterpret_cast<const AnyVec *>(src)[i];
            d[4 * i] = v.x; d[4 * i + 1] = v.y; d[4 * i + 2] = v.z; d[4 * i + 3] = v.w;
        }
    } else if (!WHOLE && K >= 4) {
        const int last = (int)(K - 4 - k0);  // of the row's last whole dword, from src on: above -512 - 4, below 4 NW
#pragma unroll
        for (int i = 0; i < NW; ++i) d[i] = reinterpret_cast<const AnyWord *>(src + (4 * i < last ? 4 * i : last))->x;
#pragma unroll
        for (int i = 0; i < NW; ++i) {
            const int past = 4 * i - last;  // codes of the clamped dword that lie before position k0 + 4 i
            const int shift = past <= 0 ? 0 : past >= 4 ? 32 : 8 * past;
            d[i] = (uint32_t)((d[i] | 0xffffffff00000000ull) >> shift);
        }
    } else {
#pragma unroll
        for (int i = 0; i < NW; ++i) d[i] = 0xffffffffu;
        if (!WHOLE && k0 == 0)
            for (int k = 0; k < (int)K; ++k) d[0] ^= (uint32_t)(src[k] ^ 0xffu) << (8 * k);
    }
}

// Packs one 32-element group kg of a row: d[2t + jh] = the four codes 8t + 4jh + (0..3), one per byte,
// already masked to `bits` bits.  Adds the codes to `sum`.  The four lanes 4x .. 4x+3 of a wave must hold
// the four groups ks = 0..3 of one k block and call this together (single groups exchange words).
// `flip`: top bit of every byte for a row of an 8-bit operand that exists (signed bytes), else 0.
__device__ __forceinline__ void pack_group(uint32_t *__restrict__ packed, int64_t row, int64_t nkb, int bits,
                                           int64_t kg, const uint32_t (&d)[8], uint32_t flip, uint32_t &sum)
{
#pragma unroll
    for (int t4 = 0; t4 < 8; ++t4) sum = __builtin_amdgcn_sad_u8(d[t4], 0u, sum);  // + the four bytes
    const int64_t kb = kg / kWordsPerRow;
    const int ks = (int)(kg % kWordsPerRow);
    if (byte_form(bits)) {
        uint4 *dst = reinterpret_cast<uint4 *>(packed + tile_row_word(row, kb, nkb, bits, 2 * ks));
        dst[0] = make_uint4(d[0] ^ flip, d[1] ^ flip, d[2] ^ flip, d[3] ^ flip);
        dst[kPlaneWords / 4] = make_uint4(d[4] ^ flip, d[5] ^ flip, d[6] ^ flip, d[7] ^ flip);
        return;
    }
    if (nibble_form(bits))
        *reinterpret_cast<uint4 *>(packed + tile_row_word(row, kb, nkb, bits, ks)) =
            make_uint4(nibble_word(d[0], d[1]), nibble_word(d[2], d[3]), nibble_word(d[4], d[5]), nibble_word(d[6], d[7]));
    for (int h = first_pair_group(bits); h < pair_groups(bits); ++h) {
        // S[2 ks + tp], tp = 0, 1: slot 2h + ks/2, words 2 (ks % 2) + tp
        uint32_t s[2];
#pragma unroll
        for (int tp = 0; tp < 2; ++tp) {
            uint32_t word = 0;
#pragma unroll
            for (int tt = 0; tt < 2; ++tt)
#pragma unroll
                for (int jh = 0; jh < 2; ++jh)
                    word |= ((d[2 * (2 * tp + tt) + jh] >> (2 * h)) & 0x03030303u) << (4 * jh + 2 * tt);
            s[tp] = word;
        }
        uint32_t *dst = packed + tile_row_word(row, kb, nkb, bits, 2 * h + (ks >> 1)) + 2 * (ks & 1);
        *reinterpret_cast<uint2 *>(dst) = make_uint2(s[0], s[1]);
    }
    if (has_single_group(bits)) {
        uint32_t l[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            uint32_t word = 0;
#pragma unroll
            for (int jh = 0; jh < 2; ++jh) word |= ((d[2 * t + jh] >> (bits - 1)) & 0x01010101u) << (4 * jh);
            word <<= ks;
            word |= __shfl_xor(word, 1);
            word |= __shfl_xor(word, 2);
            l[t] = word;
        }
        // every lane of the four now holds L[0..3]; lane ks stores L[ks]
        const uint32_t mine = ks == 0 ? l[0] : ks == 1 ? l[1] : ks == 2 ? l[2] : l[3];
        packed[tile_row_word(row, kb, nkb, bits, bits - 1) + ks] = mine;
    }
}

// The same for the field form of 3- and 4-bit activations (apmm_layout.h): the 32 codes of the group
// become the 192-bit E2M3 operand of k step ks, field 8 t + 2 c + jh at bit 6 (8 t + 2 c + jh).
__device__ __forceinline__ uint64_t spread_bytes_12(uint32_t x)
{
    // byte c of x -> bits 12 c .. 12 c + 7
    return (uint64_t)((x & 0xffu) | ((x & 0xff00u) << 4) | ((x & 0xff0000u) << 8)) | ((uint64_t)(x >> 24) << 36);
}

// words 6 ks .. 6 ks + 5 of the row's 24: slot w / 4, word w % 4
__device__ __forceinline__ void store_fields(uint32_t *__restrict__ packed, int64_t row, int64_t nkb, int64_t kg,
                                             const uint32_t (&dw)[6])
{
    const int64_t kb = kg / kWordsPerRow;
    const int ks = (int)(kg % kWordsPerRow);
    uint32_t *base = packed + tile_row_word(row, kb, nkb, 6, 0) + 3 * (ks >> 1) * kPlaneWords;
    if ((ks & 1) == 0) {
        *reinterpret_cast<uint4 *>(base) = make_uint4(dw[0], dw[1], dw[2], dw[3]);
        *reinterpret_cast<uint2 *>(base + kPlaneWords) = make_uint2(dw[4], dw[5]);
    } else {
        *reinterpret_cast<uint2 *>(base + kPlaneWords + 2) = make_uint2(dw[0], dw[1]);
        *reinterpret_cast<uint4 *>(base + 2 * kPlaneWords) = make_uint4(dw[2], dw[3], dw[4], dw[5]);
    }
}

// pack_rows_kernel: one wave per row: lane l packs the 32-element groups l, l+64, ... (two 16-byte loads of codes
// each, 1 KB contiguous per load instruction) and keeps a running code sum; the wave adds the 64 partial sums
// with lane permutes (over_wave).  Reads are ideal, writes are 8- and 16-byte pieces that other waves complete to whole
// lines later.  Used for group-form operands of one or two bits, where little is written, but for the largest (rule:
// pack_by_eights).
template <int bits, bool WHOLE>
__global__ __launch_bounds__(kThreads) void pack_rows_kernel(const uint8_t *__restrict__ codes, int64_t rows,
                                                        int64_t K, uint32_t *__restrict__ packed,
                                                        int64_t rows_p, int64_t nkb)
{
    const int lane = threadIdx.x & 63;
    const int64_t row = (int64_t)blockIdx.x * kRowsPerWg + wave_of_workgroup();
    if (row >= rows_p) return;
    const int64_t groups = nkb * kWordsPerRow;  // 32-element groups per row, a multiple of 16
    const uint32_t code_mask = 0x01010101u * ((1u << bits) - 1u);
    uint32_t sum = 0;                           // sum of the codes of this lane's groups

    auto load_group = [&](int64_t kg, uint32_t (&d)[8]) __attribute__((always_inline)) {
        if (row < rows) {
            load_codes<WHOLE>(codes + row * K, K, kg * 32, d);
#pragma unroll
            for (int t4 = 0; t4 < 8; ++t4) d[t4] &= code_mask;
        } else {
#pragma unroll
            for (int t4 = 0; t4 < 8; ++t4) d[t4] = 0u;
        }
    };

    // two groups per lane and pass, both loaded before either is packed (more bytes in flight);
    // groups is a multiple of 16, so the lanes 4x .. 4x+3 always take the same branch
    for (int64_t kg = lane; kg < groups; kg += 128) {
        uint32_t d0[8], d1[8];
        const bool second = kg + 64 < groups;
        load_group(kg, d0);
        if (second) load_group(kg + 64, d1);
        pack_group(packed, row, nkb, bits, kg, d0, 0u, sum);
        if (second) pack_group(packed, row, nkb, bits, kg + 64, d1, 0u, sum);
    }
    sum = sum_over_wave(sum);
    if (lane == 0) packed[row_sum_word(rows_p, nkb, bits) + row] = sum;
}

// pack_kernel: one wave per packed tile (32 rows x 128 k), plus one wave per row for the code sums.
//   Tile wave: lane l takes row l % 32 of the tile and the 64 codes of k steps 2h, 2h + 1, h = l / 32 (four
//   16-byte loads; the two lanes of a row read one 128-byte line between them).  What it writes is whole
//   16-byte vectors of a slot: a pair group gives S[4h .. 4h + 3] = one vector of slot 2 g + h, the field form
//   words 12h .. 12h + 11 = three vectors, a single group L[0 .. 3] after one exchange with the lane of the other
//   half.  The 32 lanes of a half write 512 contiguous bytes per vector, and consecutive waves consecutive
//   tiles: every cache line is written whole by one instruction.  (A wave per row, the earlier form, wrote
//   16-byte pieces 512 bytes apart, which other waves completed later: 1.8 TB/s for 4-bit activations where this
//   form reaches the bandwidth of the copy.)
//   Sum wave: adds the codes of one row and the padding; the sum waves of a row block follow its tile waves in
//   the grid, so that they find the rows in L2.
constexpr int kRowBlocksPerZ = 32768;  // size of the grid's y where z is needed
enum PackForm { kFieldForm, kFold3, kFold4, kByteForm, kOtherForm };  // compile-time: a launch fetches the code of its own form only

// The 64 codes of k steps 2h, 2h + 1 of row r of a tile (the tile'th of the operand), d[e][2t + jh] = the four codes 8t + 4jh + (0..3) of k step 2h + e,
// one per byte and masked: packed and stored.  The lane of the other half of the row's k block is lane ^ PARTNER.
template <PackForm FORM, int PARTNER>
__device__ __forceinline__ void pack_half_block(uint32_t *__restrict__ packed, int64_t tile, int bits, int r, int h, bool exists, const uint32_t (&d)[2][8])
{
            constexpr int kSlotVec = kPlaneWords / 4;
            // word 0 of the lane's row in a slot of the tile
            auto slot_of = [&](int n, int slot) __attribute__((always_inline)) { return packed + tile * (n * kPlaneWords) + (uint32_t)(slot * kPlaneWords + r * kWordsPerRow); };
            if constexpr (FORM == kFieldForm || FORM == kFold3 || FORM == kFold4) {
                // k step ks: words 6 ks .. 6 ks + 5 of the row's 24, the 32 codes as 6-bit fields, field 8t + 2c + jh
                uint32_t dw[12];
    #pragma unroll
                for (int e = 0; e < 2; ++e) {
                    uint64_t chunk[4];  // the 48 bits of t = 0..3
    #pragma unroll
                    for (int t = 0; t < 4; ++t)
                        chunk[t] = spread_bytes_12(d[e][2 * t]) | (spread_bytes_12(d[e][2 * t + 1]) << 6);
                    dw[6 * e + 0] = (uint32_t)chunk[0];
                    dw[6 * e + 1] = (uint32_t)(chunk[0] >> 32) | ((uint32_t)chunk[1] << 16);
                    dw[6 * e + 2] = (uint32_t)(chunk[1] >> 16);
                    dw[6 * e + 3] = (uint32_t)chunk[2];
                    dw[6 * e + 4] = (uint32_t)(chunk[2] >> 32) | ((uint32_t)chunk[3] << 16);
                    dw[6 * e + 5] = (uint32_t)(chunk[3] >> 16);
                }
                if constexpr (FORM == kFold4) {
                    uint4 *dst = reinterpret_cast<uint4 *>(slot_of(4, 2 * h));
    #pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        const uint32_t f[6] = {dw[6 * e], dw[6 * e + 1], dw[6 * e + 2], dw[6 * e + 3], dw[6 * e + 4], dw[6 * e + 5]};
                        uint32_t w[4];
                        fold_words<4>(f, w);
                        dst[e * kSlotVec] = make_uint4(w[0], w[1], w[2], w[3]);
                    }
                    return;
                }
                if constexpr (FORM == kFold3) {  // pair words of both k steps = slot h; top words 2 h, 2 h + 1 of slot 2
                    uint32_t w[2][3];
    #pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        const uint32_t f[6] = {dw[6 * e], dw[6 * e + 1], dw[6 * e + 2], dw[6 * e + 3], dw[6 * e + 4], dw[6 * e + 5]};
                        fold_words<3>(f, w[e]);
                    }
                    uint32_t *dst = slot_of(3, 0);
                    *reinterpret_cast<uint4 *>(dst + h * kPlaneWords) = make_uint4(w[0][0], w[0][1], w[1][0], w[1][1]);
                    *reinterpret_cast<uint2 *>(dst + 2 * kPlaneWords + 2 * h) = make_uint2(w[0][2], w[1][2]);
                    return;
                }
                uint4 *dst = reinterpret_cast<uint4 *>(slot_of(6, 3 * h));
    #pragma unroll
                for (int v = 0; v < 3; ++v) dst[v * kSlotVec] = make_uint4(dw[4 * v], dw[4 * v + 1], dw[4 * v + 2], dw[4 * v + 3]);
            } else if constexpr (FORM == kByteForm) {
                const uint32_t flip = exists ? 0x80808080u : 0u;
                uint4 *dst = reinterpret_cast<uint4 *>(slot_of(bits, 4 * h));
    #pragma unroll
                for (int e = 0; e < 2; ++e)
    #pragma unroll
                    for (int tp = 0; tp < 2; ++tp)
                        dst[(2 * e + tp) * kSlotVec] = make_uint4(d[e][4 * tp] ^ flip, d[e][4 * tp + 1] ^ flip, d[e][4 * tp + 2] ^ flip,
                                                                  d[e][4 * tp + 3] ^ flip);
            } else {
                if (nibble_form(bits)) {
                    uint4 *dst = reinterpret_cast<uint4 *>(slot_of(bits, 2 * h));
    #pragma unroll
                    for (int e = 0; e < 2; ++e)
                        dst[e * kSlotVec] = make_uint4(nibble_word(d[e][0], d[e][1]), nibble_word(d[e][2], d[e][3]),
                                                       nibble_word(d[e][4], d[e][5]), nibble_word(d[e][6], d[e][7]));
                }
                for (int g = first_pair_group(bits); g < pair_groups(bits); ++g) {
                    // S[2 ks + tp] of k steps 2h, 2h + 1 = S[4h .. 4h + 3] = slot 2 g + h
                    uint32_t sw[4];
    #pragma unroll
                    for (int e = 0; e < 2; ++e)
    #pragma unroll
                        for (int tp = 0; tp < 2; ++tp) {
                            uint32_t word = 0;
    #pragma unroll
                            for (int tt = 0; tt < 2; ++tt)
    #pragma unroll
                                for (int jh = 0; jh < 2; ++jh)
                                    word |= ((d[e][2 * (2 * tp + tt) + jh] >> (2 * g)) & 0x03030303u) << (4 * jh + 2 * tt);
                            sw[2 * e + tp] = word;
                        }
                    *reinterpret_cast<uint4 *>(slot_of(bits, 2 * g + h)) =
                        make_uint4(sw[0], sw[1], sw[2], sw[3]);
                }
                if (has_single_group(bits)) {
                    // L[t]: the top bit of element (ks, t, jh, c) at bit 8c + 4jh + ks; the two halves hold two k steps each
                    uint32_t l[4];
    #pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        uint32_t word = 0;
    #pragma unroll
                        for (int e = 0; e < 2; ++e)
    #pragma unroll
                            for (int jh = 0; jh < 2; ++jh)
                                word |= (((d[e][2 * t + jh] >> (bits - 1)) & 0x01010101u) << (4 * jh)) << (2 * h + e);
                        l[t] = word | __shfl_xor(word, PARTNER);
                    }
                    if (h == 0)
                        *reinterpret_cast<uint4 *>(slot_of(bits, bits - 1)) =
                            make_uint4(l[0], l[1], l[2], l[3]);
                }
            }
}

template <PackForm FORM, bool WHOLE>
__global__ __launch_bounds__(kThreads, 8) void pack_kernel(const uint8_t *__restrict__ codes, int64_t rows,
                                                        int64_t K, int bits, uint32_t *__restrict__ packed,
                                                        int64_t rows_p, int64_t nkb)
{
    const int lane = threadIdx.x & 63;
    // jobs of a row block: its nkb tiles, then the sums of its 32 rows (which find the rows in L2); a row block to each blockIdx.y and z
    const int64_t j = (int64_t)blockIdx.x * kRowsPerWg + wave_of_workgroup();
    const int64_t rb = (int64_t)blockIdx.z * kRowBlocksPerZ + blockIdx.y;
    if (rb >= rows_p / kRowBlock) return;
    const uint32_t code_mask = 0x01010101u * ((1u << bits) - 1u);
    if (j < nkb) {
        const int64_t kb = j;
        const int r = lane & 31, h = lane >> 5;
        const int64_t row = rb * kRowBlock + r;
        // d[e][2t + jh] = the four codes 8t + 4jh + (0..3) of k step 2h + e, one per byte
        uint32_t d[2][8];
        if (row < rows) {
            uint32_t v[16];
            load_codes<WHOLE>(codes + rb * kRowBlock * K + r * K, K, kb * kKBlock + 64 * h, v);
#pragma unroll
            for (int i = 0; i < 16; ++i) d[i >> 3][i & 7] = v[i] & code_mask;
        } else {
#pragma unroll
            for (int i = 0; i < 16; ++i) d[i >> 3][i & 7] = 0u;  // rows past the operand are zero words
        }
        pack_half_block<FORM, 32>(packed, rb * nkb + kb, bits, r, h, row < rows, d);
    } else {
        const int64_t row = rb * kRowBlock + (j - nkb);
        uint32_t sum = 0;
        if (row < rows) {
            const uint8_t *src = codes + row * K;
            const int64_t vecs = K / 16;
            // Eight loads under way, past the end the last vector's again: a loop that is only unrolled ends in single steps, each a round trip to
            // memory, and 5120 codes were nothing but its end (four bits 512 x 5120 4.1 -> 3.4 us, 512 x 13824 6.4 -> 5.0).  The last 4096 codes one by
            // one: their tile waves are not much longer, and loads that go ahead of the tiles' cost more where there are many rows (2048 x 4096 5.3 us,
            // this way 5.2, four at a time 5.7).
            int64_t i0 = 0;
            auto step = [&](auto u_c, auto load) __attribute__((always_inline)) {
                constexpr int U = decltype(u_c)::value;
                uint32_t v[U][4];
                const uint32_t last = vecs - i0 > 64 * U ? 64 * U - 1 : (uint32_t)(vecs - i0) - 1;
#pragma unroll
                for (int u = 0; u < U; ++u) load(src + 16 * i0 + 16 * min(64u * u + lane, last), v[u]);
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const uint32_t mask = 64u * u + lane <= last ? code_mask : 0u;
#pragma unroll
                    for (int w = 0; w < 4; ++w) sum = __builtin_amdgcn_sad_u8(v[u][w] & mask, 0u, sum);
                }
                i0 += 64 * U;
            };
            using U1 = std::integral_constant<int, 1>;
            using U4 = std::integral_constant<int, 4>;
            using U8 = std::integral_constant<int, 8>;
            if (WHOLE || (reinterpret_cast<uintptr_t>(src) & 3u) == 0) {
                auto load = [](const uint8_t *at, uint32_t (&d)[4]) __attribute__((always_inline)) {
                    const AnyVec v = *reinterpret_cast<const AnyVec *>(at);
                    d[0] = v.x; d[1] = v.y; d[2] = v.z; d[3] = v.w;
                };
                while (vecs - i0 > 64 * 4) step(U8{}, load);
                while (i0 < vecs) step(U1{}, load);
            } else {
                auto load = [](const uint8_t *at, uint32_t (&d)[4]) __attribute__((always_inline)) { load_bytes<4>(at, d); };
                while (i0 < vecs) step(U4{}, load);
            }
            if (16 * vecs + lane < K) sum += src[16 * vecs + lane] & (code_mask & 0xffu);  // at most 15 codes
            sum = sum_over_wave(sum);
            sum += (uint32_t)(nkb * kKBlock - K) * (code_mask & 0xffu);  // the all-ones codes of the padding
        }
        if (lane == 0) packed[row_sum_word(rows_p, nkb, FORM == kFieldForm ? 6 : bits) + row] = sum;
    }
}

// pack_eights_kernel: a workgroup packs eight rows, a wave eight rows x 512 codes at a time: lane l takes row l % 8 and the 64 codes of piece l / 8.  The
// eight rows' 16 bytes of a slot are one line, written whole, as by pack_kernel, and the code sums fall out on the way: no code is read twice.  Bound by
// memory.  Launches inside a graph, codes and output in the last-level cache / from and to memory: three bits 5003 x 3001 8.7 -> 7.0 / 9.8 -> 8.3 us, four bits 11008 x 4096
// 17.1 -> 13.2 / 19.1 -> 15.9, activations of four bits 2048 x 4096 5.3 -> 4.7 / 6.0 -> 5.8, two bits 11008 x 11008 26.6 -> 24.8 / 46.8 -> 35.6 (rule: pack_by_eights).  (The four
// workgroups of a row block on one XCD, one behind the other: 0.96 - 1.09 of this.)
template <PackForm FORM, bool WHOLE>
__global__ __launch_bounds__(64 * kEightWaves) void pack_eights_kernel(const uint8_t *__restrict__ codes, int64_t rows, int64_t K, int bits,
                                                                       uint32_t *__restrict__ packed, int64_t rows_p, int64_t nkb)
{
    __shared__ uint32_t sums[kEightWaves][8];
    const int lane = threadIdx.x & 63, wave = wave_of_workgroup(), waves = (int)(blockDim.x >> 6);
    const int r = lane & 7, c = lane >> 3;
    const int64_t row0 = (int64_t)blockIdx.x * 8, rb = row0 / kRowBlock;
    const int in_block = (int)(row0 % kRowBlock) + r;
    const bool exists = row0 + r < rows;
    const uint32_t code_mask = 0x01010101u * ((1u << bits) - 1u);
    const int pieces = (int)(nkb / 4);
    uint32_t sum = 0;
    auto load = [&](int g, uint32_t (&d)[2][8]) __attribute__((always_inline)) {
        if (exists) {
            uint32_t v[16];
            load_codes<WHOLE>(codes + row0 * K + r * K, K, (int64_t)g * kKPad + 64 * c, v);
#pragma unroll
            for (int i = 0; i < 16; ++i) d[i >> 3][i & 7] = v[i] & code_mask;
        } else {
#pragma unroll
            for (int i = 0; i < 16; ++i) d[i >> 3][i & 7] = 0u;  // rows past the operand are zero words
        }
    };
    for (int g = wave; g < pieces; g += waves) {
        uint32_t d[2][8];
        load(g, d);
#pragma unroll
        for (int i = 0; i < 16; ++i) sum = __builtin_amdgcn_sad_u8(d[i >> 3][i & 7], 0u, sum);
        pack_half_block<FORM, 8>(packed, rb * nkb + 4 * g + (c >> 1), bits, in_block, c & 1, exists, d);
    }
    sum += __shfl_xor(sum, 8);
    sum += __shfl_xor(sum, 16);
    sum += __shfl_xor(sum, 32);
    if (lane < 8) sums[wave][lane] = sum;
    __syncthreads();
    if (threadIdx.x < 8) {
        sum = 0;
        for (int w = 0; w < waves; ++w) sum += sums[w][lane];
        packed[row_sum_word(rows_p, nkb, FORM == kFieldForm ? 6 : bits) + row0 + lane] = sum;
    }
}

// Fused quantise + pack (paper Sec. 3.1: the feature matrix is quantised onto the symmetric bipolar-INT
// grid; Sec. 4.1: decomposition and reassembly).  One to sixteen waves per row (token; rule: quantize_waves):
//   1. max |x| over the row (on the bit patterns, two halves per operation);
//      scale = half(max|x| / (2^bits - 1)), stored per token; r = 1 / scale;
//   2. u = clamp(floor(x / (2 scale)) + 2^(bits-1), 0, 2^bits - 1): x / scale moved to the nearest odd
//      integer (ties upward), as a code; the floor is that of the exact quotient (computed as x * (r / 2)
//      with a correction that covers the rounding of r and of the product); then the same packing as pack_kernel.
// Up to 4096 elements for each wave stay in registers between the two steps; what is beyond is read again (from
// L2).  The codes are those of exact arithmetic on the binary16 inputs and the binary16 scale.  A row whose
// scale rounds to zero gets the code of +1 everywhere.
//
// WAVES waves of a workgroup share a row, one 32-element group per lane and step, so that a row takes one or two round
// trips to memory however long it is.  With one wave per row, the earlier form, a lane worked through up to eleven groups
// in turn.  Four bits, one launch inside a graph: 16 x 5120 6.0 -> 3.2 us, 16 x 13824 12.5 -> 4.1 us (4.0 with eight waves), 1024 x 11008 15.1 ->
// 13.0 us; two bits 4096 x 4096 12.5 -> 10.0 us.  Large matrices in the field form are bound by their scattered stores: those go to
// quantize_fields_kernel.
// The eight rows that share the 128-byte lines of a slot are packed on one XCD, whose L2 joins their 16-byte pieces.
typedef unsigned short us2 __attribute__((ext_vector_type(2)));
constexpr int kCachedGroups = 2;  // 32-element groups per lane kept in registers

// h[i] = elements 2i, 2i+1 of group kg as two binary16 bit patterns; elements past K read as +0
template <bool WHOLE>
__device__ __forceinline__ void load_halves(const uint16_t *xrow, int64_t K, int64_t kg, uint32_t (&h)[16])
{
    const int64_t k0 = kg * 32;
    if (!WHOLE && k0 + 32 <= K && ((2 * K | (int64_t)reinterpret_cast<uintptr_t>(xrow)) & 3) != 0) {
        load_bytes<16>(xrow + k0, h);
    } else if (k0 + 32 <= K) {
        const AnyVec *src = reinterpret_cast<const AnyVec *>(xrow + k0);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const AnyVec q = src[v];
            h[4 * v] = q.x; h[4 * v + 1] = q.y; h[4 * v + 2] = q.z; h[4 * v + 3] = q.w;
        }
    } else if (!WHOLE && K >= 2) {  // the row's end: dwords clamped to the last two elements, those before position k shifted out
        const int last = (int)(K - 2 - k0);
#pragma unroll
        for (int i = 0; i < 16; ++i) h[i] = reinterpret_cast<const AnyWord *>(xrow + k0 + (2 * i < last ? 2 * i : last))->x;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int past = 2 * i - last;
            h[i] = past <= 0 ? h[i] : past == 1 ? h[i] >> 16 : 0u;
        }
    } else {
#pragma unroll
        for (int i = 0; i < 16; ++i) h[i] = 0u;
        if (!WHOLE && kg == 0) h[0] = xrow[0];
    }
}

__device__ __forceinline__ us2 fold_max(us2 m, const uint32_t (&h)[16])
{
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const uint32_t mag = h[i] & 0x7fff7fffu;  // |x| orders like its bit pattern
        m = __builtin_elementwise_max(m, us2{(unsigned short)(mag & 0xffffu), (unsigned short)(mag >> 16)});
    }
    return m;
}

// The grid of a row from its largest magnitude
struct Grid {
    float half_r, mid, top;
    uint16_t scale;
    __device__ __forceinline__ Grid(uint32_t max_bits, int bits)
    {
        const float amax = __half2float(__ushort_as_half((uint16_t)max_bits));
        mid = (float)(1u << (bits - 1));
        top = (float)((1u << bits) - 1u);
        const __half sh = __float2half_rn(amax / top);
        const float s = __half2float(sh);
        scale = __half_as_ushort(sh);
        half_r = s > 0.0f ? (1.0f / s) * 0.5f : 0.0f;  // scale 0: every code becomes 2^(bits-1)
    }
    // code of element i of a group as a float
    __device__ __forceinline__ float code(const uint32_t (&h)[16], int i) const
    {
        const uint32_t pair = h[i >> 1];
        const float xf = __half2float(__ushort_as_half((uint16_t)((i & 1) ? pair >> 16 : pair & 0xffffu)));
        // t = x / (2 s) up to 2^-23 relative (rounded reciprocal, rounded product); the cell is floor of
        // the exact quotient.  An exact quotient that is an integer c (x on a border, ties upward) may
        // come out just below c; any other exact quotient is at least 2^-12 away from every integer
        // (x and 2 c s are binary16 numbers times small integers), and |t| <= 129.  Moving t up by
        // 2^-21 |t| (between 2^-23 |t| and 2^-12) therefore gives the exact floor in every case.
        const float t = fmaf(xf, half_r, 0.0f);  // the rounded product, with the conversion of xf in the same instruction
        const float u = floorf(fmaf(fabsf(t), 0x1p-21f, t)) + mid;  // exact: |floor| is far below 2^24
        return __builtin_amdgcn_fmed3f(u, 0.0f, top);
    }
};

// The six field words of group kg from its halves h (elements past K: the all-ones padding code); adds the codes to `sum`.
// Four fields of six bits make an integer below 2^24, which a float holds: three fused multiply-adds and one conversion for four
// codes, and the group's code sum.
template <bool WHOLE>
__device__ __forceinline__ void quantize_fields(const Grid &grid, int64_t K, int64_t kg, const uint32_t (&h)[16], uint32_t &sum, uint32_t (&dw)[6])
{
    const bool whole = WHOLE || kg * 32 + 32 <= K;
    auto code = [&](int i) __attribute__((always_inline)) { return !whole && kg * 32 + i >= K ? grid.top : grid.code(h, i); };
    uint32_t quad[8];
    float total = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {  // fields 4 i .. 4 i + 3: elements c = 2 (i % 2), 2 (i % 2) + 1, jh = 0, 1 of t = i / 2
        const int at = 8 * (i >> 1) + 2 * (i & 1);
        const float u0 = code(at), u1 = code(at + 4), u2 = code(at + 1), u3 = code(at + 5);
        total += (u0 + u1) + (u2 + u3);
        quad[i] = (uint32_t)fmaf(u3, 262144.f, fmaf(u2, 4096.f, fmaf(u1, 64.f, u0)));
    }
    sum += (uint32_t)total;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        dw[3 * i] = quad[4 * i] | (quad[4 * i + 1] << 24);
        dw[3 * i + 1] = (quad[4 * i + 1] >> 8) | (quad[4 * i + 2] << 16);
        dw[3 * i + 2] = (quad[4 * i + 2] >> 16) | (quad[4 * i + 3] << 8);
    }
}
// The same of a group of padding (every plane bit set), or zero words for a padding row
__device__ __forceinline__ void fill_fields(uint32_t fill, uint32_t &sum, uint32_t (&dw)[6])
{
    const uint32_t quad = fill * 0x41041u;
    dw[0] = dw[3] = quad | (quad << 24);
    dw[1] = dw[4] = (quad >> 8) | (quad << 16);
    dw[2] = dw[5] = (quad >> 16) | (quad << 8);
    sum += 32u * fill;
}

constexpr int quantize_threads(int waves) { return waves > kThreads / 64 ? 64 * waves : kThreads; }
template <int WAVES, bool WHOLE, bool FIELD>
__device__ __forceinline__ void quantize_rows(const uint16_t *__restrict__ x, int64_t rows, int64_t K, int bits, uint32_t *__restrict__ packed,
                                              uint16_t *__restrict__ scale_out, int64_t rows_p, int64_t nkb)
{
    constexpr int THREADS = quantize_threads(WAVES), T = 64 * WAVES, ROWS = THREADS / T, C = 8 / ROWS;  // threads of a row, rows of a workgroup, workgroups of eight rows
    const int tid = threadIdx.x % T, sub = wave_of_workgroup() / WAVES;
    const int xcd = blockIdx.x % 8, turn = blockIdx.x / 8;  // workgroups go to the XCDs in turn
    const int64_t row = (((int64_t)(turn / C) * 8 + xcd) * C + turn % C) * ROWS + sub;
    if (row >= rows_p) return;  // (rows_p is a multiple of ROWS: the whole workgroup leaves)
    const int64_t groups = nkb * kWordsPerRow;
    const uint16_t *xrow = x + row * K;

    const bool live = row < rows;
    const int64_t live_groups = live ? (K + 31) / 32 : 0;  // groups that hold at least one element
    uint32_t cache[kCachedGroups][16];
    us2 m2 = {0, 0};
#pragma unroll
    for (int it = 0; it < kCachedGroups; ++it) {
        const int64_t kg = tid + T * it;
        if (kg < live_groups) {
            load_halves<WHOLE>(xrow, K, kg, cache[it]);
            m2 = fold_max(m2, cache[it]);
        }
    }
    for (int64_t kg = tid + T * kCachedGroups; kg < live_groups; kg += T) {
        uint32_t h[16];
        load_halves<WHOLE>(xrow, K, kg, h);
        m2 = fold_max(m2, h);
    }
    uint32_t mbits = m2[0] > m2[1] ? m2[0] : m2[1];
    mbits = max_over_wave(mbits);
    __shared__ uint32_t joint[2][THREADS / 64];
    if constexpr (WAVES > 1) {
        if ((threadIdx.x & 63) == 0) joint[0][threadIdx.x / 64] = mbits;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            const uint32_t o = joint[0][sub * WAVES + w];
            mbits = o > mbits ? o : mbits;
        }
    }
    const Grid grid(mbits, bits);
    if (live && tid == 0) scale_out[row] = grid.scale;

    const uint32_t flip = byte_form(bits) && live ? 0x80808080u : 0u;
    uint32_t sum = 0;
    // codes of group kg from its halves h (elements past K: the all-ones padding code), then the packing
    auto quantize_group = [&](int64_t kg, const uint32_t (&h)[16]) __attribute__((always_inline)) {
        if constexpr (FIELD) {
            uint32_t dw[6];
            quantize_fields<WHOLE>(grid, K, kg, h, sum, dw);
            store_fields(packed, row, nkb, kg, dw);
        } else {
            const bool whole = WHOLE || kg * 32 + 32 <= K;
            auto code = [&](int i) __attribute__((always_inline)) { return !whole && kg * 32 + i >= K ? grid.top : grid.code(h, i); };
            uint32_t d[8];
#pragma unroll
            for (int t4 = 0; t4 < 8; ++t4) {
                d[t4] = 0;
#pragma unroll
                for (int c = 0; c < 4; ++c) d[t4] = __builtin_amdgcn_cvt_pk_u8_f32(code(4 * t4 + c), c, d[t4]);  // byte c = u
            }
            pack_group(packed, row, nkb, bits, kg, d, flip, sum);
        }
    };
    auto fill_group = [&](int64_t kg) __attribute__((always_inline)) {
        // a whole group of padding (every plane bit set) or a padding row (zero words)
        const uint32_t fill = live ? (1u << bits) - 1u : 0u;
        if constexpr (FIELD) {
            uint32_t dw[6];
            fill_fields(fill, sum, dw);
            store_fields(packed, row, nkb, kg, dw);
        } else {
            uint32_t d[8];
#pragma unroll
            for (int t4 = 0; t4 < 8; ++t4) d[t4] = 0x01010101u * fill;
            pack_group(packed, row, nkb, bits, kg, d, flip, sum);
        }
    };
    // The four lanes that pack a k block together must take the same call: a k block with any live group
    // quantises all four of its groups (elements past K become padding codes inside quantize_group).
    const int64_t live_blocks4 = (live_groups + 3) / 4 * 4;
#pragma unroll
    for (int it = 0; it < kCachedGroups; ++it) {
        const int64_t kg = tid + T * it;
        if (kg < live_blocks4) {
            if (kg >= live_groups) {
#pragma unroll
                for (int i = 0; i < 16; ++i) cache[it][i] = 0u;
            }
            quantize_group(kg, cache[it]);
        } else if (kg < groups) {
            fill_group(kg);
        }
    }
    for (int64_t kg = tid + T * kCachedGroups; kg < groups; kg += T) {
        if (kg < live_blocks4) {
            uint32_t h[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) h[i] = 0u;
            if (kg < live_groups) load_halves<WHOLE>(xrow, K, kg, h);
            quantize_group(kg, h);
        } else {
            fill_group(kg);
        }
    }
    sum = sum_over_wave(sum);
    if constexpr (WAVES > 1) {
        if ((threadIdx.x & 63) == 0) joint[1][threadIdx.x / 64] = sum;
        __syncthreads();
        sum = 0;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) sum += joint[1][sub * WAVES + w];
    }
    if (tid == 0) packed[row_sum_word(rows_p, nkb, FIELD ? 6 : bits) + row] = sum;
}

template <int WAVES, bool WHOLE, bool FIELD>
__global__ __launch_bounds__(kThreads) void quantize_pack_kernel(const uint16_t *__restrict__ x, int64_t rows, int64_t K, int bits,
                                                                 uint32_t *__restrict__ packed, uint16_t *__restrict__ scale_out, int64_t rows_p, int64_t nkb)
{
    quantize_rows<WAVES, WHOLE, FIELD>(x, rows, K, bits, packed, scale_out, rows_p, nkb);
}
// Rows beyond 8192 elements, eight or sixteen waves to a row: a lane's groups, one behind the other, were what a few rows took their time for (rule and
// figures: quantize_waves).
template <int WAVES, bool WHOLE, bool FIELD>
__global__ __launch_bounds__(64 * WAVES) void quantize_long_kernel(const uint16_t *__restrict__ x, int64_t rows, int64_t K, int bits,
                                                                   uint32_t *__restrict__ packed, uint16_t *__restrict__ scale_out, int64_t rows_p, int64_t nkb)
{
    quantize_rows<WAVES, WHOLE, FIELD>(x, rows, K, bits, packed, scale_out, rows_p, nkb);
}

// The same for the field form of many rows: the words of four rows meet in LDS and are written in runs of 64 bytes (a slot of four rows),
// where the kernel above writes pieces of 16 and 8 bytes, 3 KB apart.  Those pieces were what bound it: 1024 x 11008 13.1 us, without
// its stores 8.8.  Eight waves to a workgroup, two to a row; a row stays in registers (GROUPS of 32 elements to a lane).
constexpr int kQuantRows = 4;
constexpr int kQuantThreads = kQuantRows * kQuantLanes;
constexpr int kQuantBlockWords = 6 * kQuantRows * kWordsPerRow + kWordsPerRow;  // a k block in LDS, with 16 bytes against bank conflicts
template <int GROUPS, bool WHOLE>
__global__ __launch_bounds__(kQuantThreads) void quantize_fields_kernel(const uint16_t *__restrict__ x, int64_t rows, int64_t K, int bits,
                                                                        uint32_t *__restrict__ packed, uint16_t *__restrict__ scale_out,
                                                                        int64_t rows_p, int64_t nkb)
{
    extern __shared__ __align__(16) uint32_t fields[];  // [k block][slot][row of the workgroup][word]
    __shared__ uint32_t joint[2][kQuantThreads / 64];
    constexpr int C = 8 / kQuantRows;
    const int wave = wave_of_workgroup(), sub = wave / (kQuantLanes / 64), tid = threadIdx.x % kQuantLanes;
    const int xcd = blockIdx.x % 8, turn = blockIdx.x / 8;  // the eight rows that share a 128-byte line: on one XCD
    const int64_t row0 = (((int64_t)(turn / C) * 8 + xcd) * C + turn % C) * kQuantRows, row = row0 + sub;
    if (row0 >= rows_p) return;  // (rows_p is a multiple of the workgroup's rows)
    const bool live = row < rows;
    const int groups = (int)nkb * kWordsPerRow, live_groups = live ? (int)((K + 31) / 32) : 0;
    const uint16_t *xrow = x + row * K;
    uint32_t h[GROUPS][16];
    us2 m2 = {0, 0};
#pragma unroll
    for (int it = 0; it < GROUPS; ++it) {
        const int kg = tid + kQuantLanes * it;
        if (kg < live_groups) {
            load_halves<WHOLE>(xrow, K, kg, h[it]);
            m2 = fold_max(m2, h[it]);
        }
    }
    uint32_t mbits = m2[0] > m2[1] ? m2[0] : m2[1];
    mbits = max_over_wave(mbits);
    if ((threadIdx.x & 63) == 0) joint[0][wave] = mbits;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kQuantLanes / 64; ++w) {
        const uint32_t o = joint[0][sub * (kQuantLanes / 64) + w];
        mbits = o > mbits ? o : mbits;
    }
    const Grid grid(mbits, bits);
    if (live && tid == 0) scale_out[row] = grid.scale;
    uint32_t sum = 0;
#pragma unroll
    for (int it = 0; it < GROUPS; ++it) {
        const int kg = tid + kQuantLanes * it;
        if (kg >= groups) continue;
        uint32_t dw[6];
        if (kg < live_groups) quantize_fields<WHOLE>(grid, K, kg, h[it], sum, dw);
        else fill_fields(live ? (1u << bits) - 1u : 0u, sum, dw);
        const int kb = kg / kWordsPerRow, ks = kg % kWordsPerRow;
        constexpr int slot = kQuantRows * kWordsPerRow;
        uint32_t *base = fields + kb * kQuantBlockWords + 3 * (ks >> 1) * slot + sub * kWordsPerRow;
        if ((ks & 1) == 0) {
            *reinterpret_cast<uint4 *>(base) = make_uint4(dw[0], dw[1], dw[2], dw[3]);
            *reinterpret_cast<uint2 *>(base + slot) = make_uint2(dw[4], dw[5]);
        } else {
            *reinterpret_cast<uint2 *>(base + slot + 2) = make_uint2(dw[0], dw[1]);
            *reinterpret_cast<uint4 *>(base + 2 * slot) = make_uint4(dw[2], dw[3], dw[4], dw[5]);
        }
    }
    sum = sum_over_wave(sum);
    if ((threadIdx.x & 63) == 0) joint[1][wave] = sum;
    __syncthreads();
    if (tid == 0) {
        uint32_t all = 0;
#pragma unroll
        for (int w = 0; w < kQuantLanes / 64; ++w) all += joint[1][sub * (kQuantLanes / 64) + w];
        packed[row_sum_word(rows_p, nkb, 6) + row] = all;
    }
    const int pieces = (int)nkb * 6 * kQuantRows;
    uint32_t *out = packed + tile_row_word(row0, 0, nkb, 6, 0);
    for (int i = threadIdx.x; i < pieces; i += kQuantThreads) {
        const int of_row = i % kQuantRows, slot = i / kQuantRows;  // slot of all k blocks
        const uint4 v = *reinterpret_cast<const uint4 *>(fields + slot / 6 * kQuantBlockWords + (slot % 6 * kQuantRows + of_row) * kWordsPerRow);
        *reinterpret_cast<uint4 *>(out + (int64_t)slot * kPlaneWords + of_row * kWordsPerRow) = v;
    }
}

__global__ __launch_bounds__(kThreads) void unpack_kernel(const uint32_t *__restrict__ packed, int64_t rows,
                                                          int64_t K, int bits, uint8_t *__restrict__ codes,
                                                          int64_t nkb, bool field)
{
    const int64_t groups = nkb * kWordsPerRow;
    const int64_t th = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (th >= rows * groups) return;
    const int64_t row = th / groups;
    const int64_t kg = th % groups;
    const int64_t kb = kg / kWordsPerRow;
    const int ks = (int)(kg % kWordsPerRow);

    uint32_t d[8];
#pragma unroll
    for (int t4 = 0; t4 < 8; ++t4) d[t4] = 0u;
    const bool folded = !field && weight_folded_form(bits);
    if (field || folded) {
        // the six field words of the k step: words 6 ks .. 6 ks + 5 of the row's 24, or folded into n words
        uint32_t dw[6];
        if (field) {
            const uint32_t *base = packed + tile_row_word(row, kb, nkb, 6, 0);
#pragma unroll
            for (int i = 0; i < 6; ++i) {
                const int w = 6 * ks + i;
                dw[i] = base[(w >> 2) * kPlaneWords + (w & 3)];
            }
        } else {
            const uint32_t *base = packed + tile_row_word(row, kb, nkb, bits, 0);
            uint32_t in[4] = {0, 0, 0, 0};
            for (int i = 0; i < bits; ++i) {
                const int w = fold_word_at(bits, ks, i);
                in[i] = base[(w >> 2) * kPlaneWords + (w & 3)];
            }
            auto word = [&](auto d_c) __attribute__((always_inline)) {
                constexpr int D = decltype(d_c)::value;
                dw[D] = bits == 4 ? unfold_word<4, D>(in[0], in[1], in[2], in[3]) : unfold_word<3, D>(in[0], in[1], in[2], 0u);
            };
            word(std::integral_constant<int, 0>{}); word(std::integral_constant<int, 1>{}); word(std::integral_constant<int, 2>{});
            word(std::integral_constant<int, 3>{}); word(std::integral_constant<int, 4>{}); word(std::integral_constant<int, 5>{});
        }
        const uint64_t chunk[4] = {(uint64_t)dw[0] | ((uint64_t)(dw[1] & 0xffffu) << 32),
                                   (uint64_t)(dw[1] >> 16) | ((uint64_t)dw[2] << 16),
                                   (uint64_t)dw[3] | ((uint64_t)(dw[4] & 0xffffu) << 32),
                                   (uint64_t)(dw[4] >> 16) | ((uint64_t)dw[5] << 16)};
        const uint32_t code_mask = (1u << bits) - 1u;
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int jh = 0; jh < 2; ++jh)
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    d[2 * t + jh] |= ((uint32_t)(chunk[t] >> (12 * c + 6 * jh)) & code_mask) << (8 * c);
    }
    if (byte_form(bits)) {
#pragma unroll
        for (int i = 0; i < 8; ++i)
            d[i] = packed[tile_row_word(row, kb, nkb, bits, 2 * ks + (i >> 2)) + (i & 3)] ^ 0x80808080u;
    }
    if (nibble_form(bits)) {
        const uint32_t *src = packed + tile_row_word(row, kb, nkb, bits, ks);
#pragma unroll
        for (int i = 0; i < 8; ++i) d[i] = (src[i >> 1] >> (4 * (i & 1))) & 0x0f0f0f0fu;
    }
    for (int h = first_pair_group(bits); !field && !folded && h < pair_groups(bits); ++h) {
        const uint32_t *src = packed + tile_row_word(row, kb, nkb, bits, 2 * h + (ks >> 1)) + 2 * (ks & 1);
#pragma unroll
        for (int tp = 0; tp < 2; ++tp) {
            const uint32_t word = src[tp];
#pragma unroll
            for (int tt = 0; tt < 2; ++tt)
#pragma unroll
                for (int jh = 0; jh < 2; ++jh)
                    d[2 * (2 * tp + tt) + jh] |= ((word >> (4 * jh + 2 * tt)) & 0x03030303u) << (2 * h);
        }
    }
    if (!field && !folded && has_single_group(bits)) {
        const uint32_t *src = packed + tile_row_word(row, kb, nkb, bits, bits - 1);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const uint32_t word = src[t] >> ks;
#pragma unroll
            for (int jh = 0; jh < 2; ++jh) d[2 * t + jh] |= ((word >> (4 * jh)) & 0x01010101u) << (bits - 1);
        }
    }
    const int64_t k0 = kg * 32;
    uint8_t *dst = codes + row * K + k0;
#pragma unroll
    for (int t4 = 0; t4 < 8; ++t4)
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if (k0 + 4 * t4 + c < K) dst[4 * t4 + c] = (uint8_t)(d[t4] >> (8 * c));
}

}  // namespace

hipError_t launch_pack(const uint8_t *codes, int64_t rows, int64_t K, int bits, bool field, uint32_t *packed,
                       hipStream_t stream)
{
    const int64_t rows_p = round_up(rows, kRowBlock);
    const int64_t nkb = round_up(K, kKPad) / kKBlock;
    if (rows_p == 0) return hipSuccess;
    const bool by_eights = pack_by_eights(rows, K, bits, field);
    if (!field && bits <= 2 && !by_eights) {
        // Row by row against tile by tile: 4096 x 4096 two-bit codes 4.7 / 6.8 us (reads in 1 KB runs, code sums on the way); four-bit activations
        // 2048 x 11008 22.6 / 12.0, where more is written.
        const int64_t blocks = (rows_p + kRowsPerWg - 1) / kRowsPerWg;
        if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
        const bool whole = K % 32 == 0;
        const auto kernel = bits == 1 ? (whole ? pack_rows_kernel<1, true> : pack_rows_kernel<1, false>)
                                      : (whole ? pack_rows_kernel<2, true> : pack_rows_kernel<2, false>);
        hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(kThreads), 0, stream, codes, rows, K, packed, rows_p, nkb);
        return hipGetLastError();
    }
    if (by_eights) {
        const bool whole = K % 64 == 0;
        const auto kernel = field ? (whole ? pack_eights_kernel<kFieldForm, true> : pack_eights_kernel<kFieldForm, false>)
                          : bits == 3 ? (whole ? pack_eights_kernel<kFold3, true> : pack_eights_kernel<kFold3, false>)
                          : bits == 4 ? (whole ? pack_eights_kernel<kFold4, true> : pack_eights_kernel<kFold4, false>)
                          : byte_form(bits) ? (whole ? pack_eights_kernel<kByteForm, true> : pack_eights_kernel<kByteForm, false>)
                                            : (whole ? pack_eights_kernel<kOtherForm, true> : pack_eights_kernel<kOtherForm, false>);
        hipLaunchKernelGGL(kernel, dim3((unsigned)(rows_p / 8)), dim3((unsigned)pack_eights_threads(K)), 0, stream, codes, rows, K, bits, packed, rows_p, nkb);
        return hipGetLastError();
    }
    // Per row block: tile waves, then sum waves (a multiple of kRowsPerWg in all).  The grid's y and z count the row blocks, so that no wave
    // divides its number.
    const int64_t blocks = (nkb + kRowBlock) / kRowsPerWg, row_blocks = rows_p / kRowBlock;
    const int64_t ny = row_blocks < kRowBlocksPerZ ? row_blocks : kRowBlocksPerZ, nz = (row_blocks + ny - 1) / ny;
    if (blocks * row_blocks > 0x7fffffffLL || nz > 32768) return hipErrorInvalidValue;
    const bool whole = K % 64 == 0;
    const auto kernel = field ? (whole ? pack_kernel<kFieldForm, true> : pack_kernel<kFieldForm, false>)
                      : bits == 3 ? (whole ? pack_kernel<kFold3, true> : pack_kernel<kFold3, false>)
                      : bits == 4 ? (whole ? pack_kernel<kFold4, true> : pack_kernel<kFold4, false>)
                      : byte_form(bits) ? (whole ? pack_kernel<kByteForm, true> : pack_kernel<kByteForm, false>)
                                        : (whole ? pack_kernel<kOtherForm, true> : pack_kernel<kOtherForm, false>);
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks, (unsigned)ny, (unsigned)nz), dim3(kThreads), 0, stream, codes, rows, K, bits, packed, rows_p, nkb);
    return hipGetLastError();
}

hipError_t launch_quantize_pack(const uint16_t *x, int64_t rows, int64_t K, int bits, bool field, uint32_t *packed,
                                uint16_t *scale, hipStream_t stream)
{
    const int64_t rows_p = round_up(rows, kRowBlock);
    const int64_t nkb = round_up(K, kKPad) / kKBlock;
    if (rows_p == 0) return hipSuccess;
    const bool whole = K % 128 == 0;  // every k block is packed whole or is all padding
    if (field && quantize_rows_by_four(rows, K)) {
        const int64_t lane_groups = quantize_lane_groups(K);
        const size_t lds = (size_t)nkb * kQuantBlockWords * 4;  // at most 51 KB
        const int64_t blocks = (rows_p / kQuantRows + 15) / 16 * 16;  // pairs for each of the eight XCDs
        if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
        auto kernel = lane_groups == 1 ? (whole ? quantize_fields_kernel<1, true> : quantize_fields_kernel<1, false>)
                    : lane_groups == 2 ? (whole ? quantize_fields_kernel<2, true> : quantize_fields_kernel<2, false>)
                    : lane_groups == 3 ? (whole ? quantize_fields_kernel<3, true> : quantize_fields_kernel<3, false>)
                                       : (whole ? quantize_fields_kernel<4, true> : quantize_fields_kernel<4, false>);
        hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(kQuantThreads), lds, stream, x, rows, K, bits, packed, scale, rows_p, nkb);
        return hipGetLastError();
    }
    const int waves = quantize_waves(rows, K, field), threads = quantize_threads(waves);
    const int64_t blocks = (rows_p + 63) / 64 * 64 * waves / (threads / 64);  // eight rows for each of the eight XCDs
    if (blocks * threads > kMostWorkItems) return hipErrorInvalidValue;
    decltype(&quantize_pack_kernel<1, true, true>) kernel;
    if (field)
        kernel = waves == 1 ? (whole ? quantize_pack_kernel<1, true, true> : quantize_pack_kernel<1, false, true>)
               : waves == 2 ? (whole ? quantize_pack_kernel<2, true, true> : quantize_pack_kernel<2, false, true>)
               : waves == 4 ? (whole ? quantize_pack_kernel<4, true, true> : quantize_pack_kernel<4, false, true>)
               : waves == 8 ? (whole ? quantize_long_kernel<8, true, true> : quantize_long_kernel<8, false, true>)
                            : (whole ? quantize_long_kernel<16, true, true> : quantize_long_kernel<16, false, true>);
    else
        kernel = waves == 1 ? (whole ? quantize_pack_kernel<1, true, false> : quantize_pack_kernel<1, false, false>)
               : waves == 2 ? (whole ? quantize_pack_kernel<2, true, false> : quantize_pack_kernel<2, false, false>)
               : waves == 4 ? (whole ? quantize_pack_kernel<4, true, false> : quantize_pack_kernel<4, false, false>)
               : waves == 8 ? (whole ? quantize_long_kernel<8, true, false> : quantize_long_kernel<8, false, false>)
                            : (whole ? quantize_long_kernel<16, true, false> : quantize_long_kernel<16, false, false>);
    const size_t lds = quantize_few_workgroups(rows, K, bits, field) ? 32000 : 0;  // not read: it leaves room for five workgroups
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3((unsigned)threads), lds, stream, x, rows, K, bits, packed, scale, rows_p, nkb);
    return hipGetLastError();
}

hipError_t launch_unpack(const uint32_t *packed, int64_t rows, int64_t K, int bits, bool field, uint8_t *codes,
                         hipStream_t stream)
{
    const int64_t nkb = round_up(K, kKPad) / kKBlock;
    const int64_t total = rows * nkb * kWordsPerRow;
    if (total == 0) return hipSuccess;
    const int64_t blocks = (total + kThreads - 1) / kThreads;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    hipLaunchKernelGGL(unpack_kernel, dim3((unsigned)blocks), dim3(kThreads), 0, stream, packed, rows, K, bits,
                       codes, nkb, field);
    return hipGetLastError();
}

}  // namespace apmm
