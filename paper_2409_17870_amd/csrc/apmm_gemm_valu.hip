// Design B: bit-plane GEMM on the vector ALU (paper Sec. 3.2 with the XOR form of the
// 1-bit product).  For planes a^(j) of the activations and w^(i) of the weights,
//   D_ij = K - 2 * popcount(a^(j) xor w^(i))        (bit 1 = +1, bit 0 = -1)
//   C    = sum_i sum_j 2^(i+j) * D_ij
//        = K * (2^p - 1)(2^q - 1) - 2 * sum_ij 2^(i+j) * popcount(a^(j) xor w^(i)).
// Padded k positions carry identical bits in both operands, so they add nothing to the
// popcounts and the true K appears in the constant.  The recovery (shift and add) is done
// in registers; nothing but C touches global memory.
//
// This kernel is the general one: any p, q in 1..8, any M, N, K.  It is the fallback for codes the
// matrix-unit kernels do not cover and the reference for design B at large M.  A workgroup of 256 threads
// owns 64 x 64 outputs, a thread 4 x 4 of them (rows ty + 16 i, columns tx + 16 j).  Per k block the
// workgroup brings every plane of its 64 + 64 rows to the same form, 16 elements per word at the even bit
// positions (in the order of apmm_layout.h or of apmm_fields.h), once, into LDS; then any activation plane can be XOR-ed with any weight plane:
// per output, plane pair and word one XOR, one popcount and one shift-and-add.  The vector ALU bounds it:
// 3 p q operations per output and 16 elements, i.e. about 0.2 effective POP/s for W1A2 if every issue slot
// of the chip did nothing else.
#include <type_traits>

#include "apmm_epilogue.h"
#include "apmm_fields.h"
#include "apmm_kernels.h"

namespace apmm {
namespace {

constexpr int kTile = 16;

// The planes of the 16 elements (ks = w / 2, tp = w % 2, all tt, jh, c) of one row and k block of an n-bit operand come from
// up to five words of the row (word x: slot x / 4, word x % 4), each read once.
constexpr int kRawWords = 5;
__device__ __forceinline__ void raw_word_places(int n, bool field_form, bool folded_form, int w, int (&x)[kRawWords])
{
    const int ks = w >> 1, tp = w & 1, single = 4 * (n - 1) + 2 * tp;  // L[2 tp] of the single group
    auto set = [&](int x0, int x1, int x2, int x3, int x4) __attribute__((always_inline)) { x[0] = x0; x[1] = x1; x[2] = x2; x[3] = x3; x[4] = x4; };
    if (field_form) set(3 * w, 3 * w + 1, 3 * w + 2, 3 * w, 3 * w);  // words 6 ks + 3 tp ...
    else if (folded_form) set(fold_word_at(n, ks, 0), fold_word_at(n, ks, 1), fold_word_at(n, ks, 2), fold_word_at(n, ks, n - 1), fold_word_at(n, ks, 0));
    else if (byte_form(n)) set(4 * w, 4 * w + 1, 4 * w + 2, 4 * w + 3, 4 * w);
    else if (nibble_form(n)) set(2 * w, 2 * w + 1, n > 5 ? 16 + w : 2 * w, n != 6 ? single : 2 * w, n != 6 ? single + 1 : 2 * w);
    else set(n == 2 ? w : single, n == 2 ? w : single + 1, n == 2 ? w : single, n == 2 ? w : single, n == 2 ? w : single);
}
// put(i, plane i) from these words.  FIELDS: in field order (apmm_fields.h), which codes stored in fields have by themselves,
// else at bits 8c + 4jh + 2tt.
template <bool FIELDS, class Put>
__device__ __forceinline__ void plane_words(const uint32_t (&raw)[kRawWords], int n, bool field_form, bool folded_form, int w, Put &&put)
{
    const int ks = w >> 1, tp = w & 1;
    auto put_pair = [&](int i, uint32_t n0, uint32_t n1) __attribute__((always_inline)) {
        const uint32_t pair = FIELDS ? join_in_field_order(n0, n1) : join_in_common_order(n0, n1);
        put(i, pair & kEvenBits);
        if (i + 1 < n) put(i + 1, (pair >> 1) & kEvenBits);
    };
    if (FIELDS && field_form) {
        for (int i = 0; i < n; ++i) put(i, field_plane(raw[0], raw[1], raw[2], i));
    } else if (FIELDS && folded_form) {
        for (int i = 0; i < n; ++i)
            put(i, n == 3 ? (tp ? folded_plane<3, 1>(raw[0], raw[1], raw[2], 0u, i) : folded_plane<3, 0>(raw[0], raw[1], raw[2], 0u, i))
                          : (tp ? folded_plane<4, 1>(raw[0], raw[1], raw[2], raw[3], i) : folded_plane<4, 0>(raw[0], raw[1], raw[2], raw[3], i)));
    } else if (byte_form(n)) {  // word 2 tt + jh: bytes with the top bit inverted
        const uint32_t f = 0x80808080u, m = 0x03030303u;
        for (int i = 0; i < 8; i += 2)
            put_pair(i, (((raw[0] ^ f) >> i) & m) | ((((raw[1] ^ f) >> i) & m) << 4), (((raw[2] ^ f) >> i) & m) | ((((raw[3] ^ f) >> i) & m) << 4));
    } else if (nibble_form(n)) {  // N[4 ks + 2 tp], N[4 ks + 2 tp + 1]; S[w] of bits 4, 5; L[2 tp], L[2 tp + 1]
        const uint32_t m = 0x33333333u;
        put_pair(0, raw[0] & m, raw[1] & m);
        put_pair(2, (raw[0] >> 2) & m, (raw[1] >> 2) & m);
        if (n > 5) put_pair(4, raw[2] & m, (raw[2] >> 2) & m);
        if (n != 6) put_pair(n - 1, (raw[3] >> ks) & 0x11111111u, (raw[4] >> ks) & 0x11111111u);
    } else if (n == 2) {
        put_pair(0, raw[0] & 0x33333333u, (raw[0] >> 2) & 0x33333333u);
    } else {
        put_pair(0, (raw[0] >> ks) & 0x11111111u, (raw[1] >> ks) & 0x11111111u);
    }
}

// plane i of words of 1- and 2-bit codes (group form), for operands that both are of these widths
__device__ __forceinline__ uint32_t group_plane_word(const uint32_t *tile_row, int n, int i, int w)
{
    if (n == 2) return (tile_row[(w >> 2) * kPlaneWords + (w & 3)] >> i) & kEvenBits;
    const uint32_t *l = tile_row + 2 * (w & 1);  // L[2 tp], L[2 tp + 1]
    return join_in_common_order((l[0] >> (w >> 1)) & 0x11111111u, (l[1] >> (w >> 1)) & 0x11111111u);
}

constexpr int kOutTile = 64;                 // outputs per workgroup and dimension
constexpr int kPerThread = kOutTile / kTile;  // outputs per thread and dimension

// NARROW: both operands of one or two bits.  A kernel of its own, because what the other forms need takes registers that
// cost it two workgroups per compute unit (2048 x 4096 x 4096 W1A1 264 -> 348 us).
template <bool NARROW>
__global__ __launch_bounds__(kTile * kTile, 4) void gemm_valu_kernel(GemmArgs g, int64_t tiles_n)
{
    // one-dimensional grid (the y dimension would cap M at about four million rows)
    const int64_t n0 = ((int64_t)blockIdx.x % tiles_n) * kOutTile, m0 = ((int64_t)blockIdx.x / tiles_n) * kOutTile;
    const int tid = threadIdx.x, tx = tid % kTile, ty = tid / kTile;
    const int p = g.p, q = g.q;
    const int64_t rows_a = round_up(g.M, kRowBlock), rows_b = round_up(g.N, kRowBlock);
    // plane words of one k block: [plane][word 0..7][row 0..63]; consecutive lanes read consecutive rows
    __shared__ uint32_t a_lds[8 * 8 * kOutTile], w_lds[8 * 8 * kOutTile];

    uint32_t weighted[kPerThread][kPerThread];  // sum_ij 2^(i+j) popcount, modulo 2^32 (the true C fits 32 bits)
#pragma unroll
    for (int i = 0; i < kPerThread; ++i)
#pragma unroll
        for (int j = 0; j < kPerThread; ++j) weighted[i][j] = 0;

    const int r = tid % kOutTile;  // (256 threads: every job of a thread is for the same row)
    // any order of the elements will do that both operands follow: field order if either has its codes in fields
    const bool field_a = activation_field_form(p), folded_w = weight_folded_form(q), fields = field_a || folded_w;

    // A thread fills word w of all planes of row r, w = tid / 64 and that + 4, of both operands; rows past an operand read its
    // last padded row.  The loads of either operand are in flight together.
    const int64_t row_a = m0 + r < rows_a ? m0 + r : rows_a - 1, row_w = n0 + r < rows_b ? n0 + r : rows_b - 1;
    auto fill = [&](auto fields_c, int64_t kb) __attribute__((always_inline)) {
        constexpr bool FIELDS = decltype(fields_c)::value;
        const uint32_t *src[2] = {g.a + tile_row_word(row_a, kb, g.nkb, activation_slots(p), 0), g.w + tile_row_word(row_w, kb, g.nkb, q, 0)};
#pragma unroll
        for (int side = 0; side < 2; ++side) {
            uint32_t raw[2][kRawWords];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                int x[kRawWords];
                raw_word_places(side ? q : p, FIELDS && !side && field_a, FIELDS && side && folded_w, tid / kOutTile + 4 * h, x);
#pragma unroll
                for (int j = 0; j < kRawWords; ++j) raw[h][j] = src[side][(x[j] >> 2) * kPlaneWords + (x[j] & 3)];
            }
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int w = tid / kOutTile + 4 * h;
                uint32_t *dst = (side ? w_lds : a_lds) + w * kOutTile + r;
                plane_words<FIELDS>(raw[h], side ? q : p, !side && field_a, side && folded_w, w,
                                    [&](int i, uint32_t v) __attribute__((always_inline)) { dst[i * 8 * kOutTile] = v; });
            }
        }
    };

    for (int64_t kb = 0; kb < g.nkb; ++kb) {
        if (kb) __syncthreads();  // every thread is done with the previous k block
        if constexpr (NARROW) {
            // one word of one plane of one row per job; rows past the operand read its last padded row
            for (int job = tid; job < (p + q) * 8 * kOutTile; job += kTile * kTile) {
                const int w = (job / kOutTile) % 8, plane = job / (8 * kOutTile);
                if (plane < p) a_lds[(plane * 8 + w) * kOutTile + r] = group_plane_word(g.a + tile_row_word(row_a, kb, g.nkb, p, 0), p, plane, w);
                else w_lds[((plane - p) * 8 + w) * kOutTile + r] = group_plane_word(g.w + tile_row_word(row_w, kb, g.nkb, q, 0), q, plane - p, w);
            }
        } else if (fields) {
            fill(std::true_type{}, kb);
        } else {
            fill(std::false_type{}, kb);
        }
        __syncthreads();
        for (int w = 0; w < 8; ++w) {
            for (int j = 0; j < p; ++j) {
                uint32_t av[kPerThread];
#pragma unroll
                for (int i = 0; i < kPerThread; ++i) av[i] = a_lds[(j * 8 + w) * kOutTile + ty + kTile * i];
                for (int i = 0; i < q; ++i) {
#pragma unroll
                    for (int jn = 0; jn < kPerThread; ++jn) {
                        const uint32_t wv = w_lds[(i * 8 + w) * kOutTile + tx + kTile * jn];
#pragma unroll
                        for (int im = 0; im < kPerThread; ++im)
                            weighted[im][jn] += (uint32_t)__popc(av[im] ^ wv) << (i + j);
                    }
                }
            }
        }
    }
    const uint32_t full = (uint32_t)g.K * (uint32_t)((1 << p) - 1) * (uint32_t)((1 << q) - 1);
#pragma unroll
    for (int im = 0; im < kPerThread; ++im) {
        const int64_t m = m0 + ty + kTile * im;
        if (m >= g.M) continue;
        const float sa = load_scale(g.a_scale, m);
#pragma unroll
        for (int jn = 0; jn < kPerThread; ++jn) {
            const int64_t n = n0 + tx + kTile * jn;
            if (n < g.N) store_output(g, m, n, (int32_t)(full - 2u * weighted[im][jn]), sa, load_scale(g.w_scale, n));
        }
    }
}

}  // namespace

hipError_t launch_gemm_valu(const GemmArgs &args, hipStream_t stream)
{
    const int64_t gx = (args.N + kOutTile - 1) / kOutTile, gy = (args.M + kOutTile - 1) / kOutTile;
    if (gx > 0x7fffffffLL / gy) return hipErrorInvalidValue;
    note_kernel("gemm_valu_kernel");
    const auto kernel = args.p <= 2 && args.q <= 2 ? gemm_valu_kernel<true> : gemm_valu_kernel<false>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)(gx * gy)), dim3(kTile * kTile), 0, stream, args, gx);
    return hipGetLastError();
}

}  // namespace apmm
