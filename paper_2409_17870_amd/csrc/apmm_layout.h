// Packed bit-plane layout shared by every kernel of the library (paper Sec. 4.1).
//
// A rows x K operand of n-bit codes is stored with n bits per element in 32-bit words, concatenated
// tile by tile:
//
//   word(rb, kb, s, r, g)   rb = row / 32       row block (rows padded to a multiple of 32)
//                           kb = k / 128        k block   (K padded to a multiple of 512: nkb is a multiple of 4)
//                           s  = plane slot, 0 .. n-1 (16 bytes per row and slot)
//                           r  = row % 32
//                           g  = word inside the slot, 0 .. 3
//   index = (((rb * nkb + kb) * n + s) * 32 + r) * 4 + g
//
// so one (rb, kb) tile is 512*n contiguous bytes and inside a slot the 32 rows are 16 bytes each:
// when the lanes of a wave take one row each, every 16-byte load instruction reads one contiguous
// 512-byte run per row block.
//
// Which bit of which word holds plane i of element k is chosen for the consumers, the matrix-unit
// kernels first.  The planes of a code are taken in groups: bits (0,1), (2,3), ... form PAIR groups,
// and when n is odd the top bit is a SINGLE group.  With the element's position inside its k block
// written as
//       k % 128 = 32*ks + 8*t + 4*jh + c,   ks, t in 0..3, jh in 0..1, c in 0..3,   t = 2*tp + tt,
//   pair group h (code bits 2h, 2h+1) fills slots 2h and 2h+1, seen as eight words S[0..7]
//       (slot 2h + w/4, word w % 4):  bit b of the group sits in S[2*ks + tp] at bit 8*c + 4*jh + 2*tt + b;
//   a single group (code bit n-1) fills slot n-1, four words L[0..3]:
//       the bit sits in L[t] at bit 8*c + 4*jh + ks.
// Reading them (apmm_mfma_common.h has the code):
//   * E2M1 (fp4) MFMA operand of k step ks: its four dwords are (S[2ks + tp] >> 2tt) & 0x33333333, i.e.
//     every nibble is 00uu with the 2-bit code of the group: 1.5 operations per dword.  For a single
//     group L[t] & (0x11111111 << ks): the bit stands at another place of the nibble in every k step,
//     which the MFMA's power-of-two operand scale undoes (1.25 operations per dword).
//   * XOR/popcount: (S[w] >> b) & 0x55555555 is plane 2h+b of 16 elements; two single-group words give
//     the same 16 elements with two shift-and-mask steps, so any two planes can be compared.
// Both operands of a GEMM use the same element -> (ks, t, jh, c) map, which is all a contraction needs.
//
// Activations of 3 or 4 bits use a second form, the FIELD form: six slots per (row, k block), i.e. 24
// words, six per k step ks (words 6 ks .. 6 ks + 5 of the row's 24, slot w / 4, word w % 4).  The 192 bits
// of a k step hold its 32 codes as 6-bit fields, field 8 t + 2 c + jh at bits 6 (8 t + 2 c + jh) ..., code in
// the low bits: exactly the E2M3 (fp6) MFMA operand of that k step, in which a 4-bit code u is the number
// u / 8.  The matrix unit multiplies fp6 and fp4 operands at the same rate, so 4-bit activations need no
// second sweep of K and no expansion at all, at the price of 6 instead of 4 bits per element in a buffer
// that lives for one GEMM.
//
// Weights of 3 or 4 bits use the FOLDED form: the same six field words F0 .. F5 per k step, folded into n words without
// losing a bit.  The fields of words 0, 1, 2 (and again 3, 4, 5) start at bit offsets 0, 4 and 2 modulo 6, so the holes of
// one word are where another has its codes, and unfolding is masks:
//   4 bits: words F0 | F4 & a, F1 | F5 & b, F2 | F4 & c, F3 | F5 & a   (a, b, c: bits 4,5 / 2,3 / 0,1 modulo 6);
//           word j of k step ks is word j of slot ks
//   3 bits: the bit pairs 0, 1 of F0, F1, F2 in one word (planes 0 and 1 at its even and odd bits), those of F3, F4, F5 in
//           another, the top bits of all six in a third (of F0 .. F2 at its even, of F3 .. F5 at its odd bits): words 2 ks,
//           2 ks + 1 of slots 0, 1 and word ks of slot 2
// Eight (4 bits) or thirteen (3 bits) operations give the E2M3 operand of 32 codes.  The two plane groups of the group
// form took twelve, and K was swept once for each: half the matrix instructions now, for the same bytes.
//
// Codes of 5 to 8 bits go to the int8 matrix operations and are stored so that little is left to do there:
//   5, 6, 7 bits: the four low bits fill slots 0 .. 3 as nibbles: word N[4 ks + t] (slot ks, word t) holds bits 0 .. 3 of element
//       (ks, t, jh, c) at bits 8c + 4jh ...; bits 4, 5 are the pair group of slots 4, 5 and the top bit of an odd width is
//       the single group of slot n - 1, both as above;
//   8 bits: bytes.  Slot 2 ks + tp, word 2 tt + jh, byte c is the code of (ks, 2 tp + tt, jh, c) with its top bit inverted, i.e.
//       u - 128 as a signed byte, in the order of the elements: the int8 operand as it stands.
//
// Behind the tiles follows one int32 per (padded) row: the sum of the row's codes over the padded K.
// The MFMA kernels multiply codes u instead of values 2u - (2^n - 1) and need these sums to recover C.
//
// Padding: elements with k >= K have every plane bit set in BOTH operands.  Their XOR is zero, and each
// contributes exactly (2^p - 1)(2^q - 1) to an integer dot product, which the kernels subtract again.
// Rows >= `rows` are all-zero words and are never stored to C.
#pragma once
#include <stdint.h>

namespace apmm {

constexpr int kRowBlock = 32;    // rows per packed tile
constexpr int kKBlock = 128;     // k elements per packed tile
constexpr int kKPad = 512;       // K is padded to a multiple of this (four k blocks = two stages of the MFMA kernel)
constexpr int kWordsPerRow = 4;  // 32-bit words per (row, slot) inside a tile
constexpr int kPlaneWords = kRowBlock * kWordsPerRow;  // words between consecutive slots of a tile

inline __host__ __device__ int64_t round_up(int64_t x, int64_t m) { return (x + m - 1) / m * m; }

// number of pair groups of an n-bit code, and whether a single group follows them
inline __host__ __device__ constexpr int pair_groups(int n) { return n / 2; }
inline __host__ __device__ constexpr bool has_single_group(int n) { return (n & 1) != 0; }

// activations of 3 or 4 bits are stored in the field form (six slots), everything else in the group form
inline __host__ __device__ constexpr bool activation_field_form(int p) { return p == 3 || p == 4; }
// codes of 5 .. 7 bits keep their four low bits as nibbles, codes of 8 bits are stored as signed bytes
inline __host__ __device__ constexpr bool nibble_form(int n) { return n >= 5 && n <= 7; }
inline __host__ __device__ constexpr bool byte_form(int n) { return n == 8; }
// first pair group that is stored as one (nibbles and bytes hold the lower bits otherwise)
inline __host__ __device__ constexpr int first_pair_group(int n) { return n <= 4 ? 0 : nibble_form(n) ? 2 : 4; }
// weights of 3 or 4 bits
inline __host__ __device__ constexpr bool weight_folded_form(int n) { return n == 3 || n == 4; }
inline __host__ __device__ constexpr int activation_slots(int p) { return activation_field_form(p) ? 6 : p; }

// Folded form: n words from the six field words of a k step (fold_words), field word D from the n words (unfold_word), and
// the place of word j of k step ks among the 4 n words of the row and k block (slot: / 4).
constexpr uint32_t kFoldBits45 = 0x30c30c30u, kFoldBits23 = 0x0c30c30cu, kFoldBits01 = 0xc30c30c3u;  // bits modulo 6
constexpr uint32_t kFoldBit0 = 0x41041041u, kFoldBit2 = 0x04104104u, kFoldBit4 = 0x10410410u;
inline __host__ __device__ constexpr int fold_word_at(int n, int ks, int j) { return n == 4 ? 4 * ks + j : j < 2 ? 2 * ks + j : 8 + ks; }
template <int N>
inline __host__ __device__ void fold_words(const uint32_t (&f)[6], uint32_t (&w)[N])
{
    static_assert(N == 3 || N == 4, "folded widths");
    if constexpr (N == 4) {
        w[0] = f[0] | (f[4] & kFoldBits45);
        w[1] = f[1] | (f[5] & kFoldBits23);
        w[2] = f[2] | (f[4] & kFoldBits01);
        w[3] = f[3] | (f[5] & kFoldBits45);
    } else {
        w[0] = (f[0] & kFoldBits01) | (f[1] & kFoldBits45) | (f[2] & kFoldBits23);
        w[1] = (f[3] & kFoldBits01) | (f[4] & kFoldBits45) | (f[5] & kFoldBits23);
        w[2] = (f[0] & kFoldBit2) | (f[1] & kFoldBit0) | (f[2] & kFoldBit4) |
               (((f[3] & kFoldBit2) | (f[4] & kFoldBit0) | (f[5] & kFoldBit4)) << 1);
    }
}
template <int N, int D>
inline __host__ __device__ uint32_t unfold_word(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t w3)
{
    static_assert((N == 3 || N == 4) && D >= 0 && D < 6, "folded widths");
    if constexpr (N == 4) {
        return D == 0 ? w0 & ~kFoldBits45 : D == 1 ? w1 & ~kFoldBits23 : D == 2 ? w2 & ~kFoldBits01 : D == 3 ? w3 & ~kFoldBits45
             : D == 4 ? (w0 & kFoldBits45) | (w2 & kFoldBits01) : (w1 & kFoldBits23) | (w3 & kFoldBits45);
    } else {
        const uint32_t pairs = D < 3 ? w0 : w1, top = D < 3 ? w2 : w2 >> 1;
        return D % 3 == 0 ? (pairs & kFoldBits01) | (top & kFoldBit2) : D % 3 == 1 ? (pairs & kFoldBits45) | (top & kFoldBit0)
                                                                                  : (pairs & kFoldBits23) | (top & kFoldBit4);
    }
}

// index of word g=0 of (row, slot s) in k block kb
inline __host__ __device__ int64_t tile_row_word(int64_t row, int64_t kb, int64_t nkb, int n, int s)
{
    int64_t rb = row / kRowBlock, r = row % kRowBlock;
    return (((rb * nkb + kb) * n + s) * kRowBlock + r) * kWordsPerRow;
}

// index of the first row-sum word: the tiles of rows_p x nkb*128 elements come first
inline __host__ __device__ int64_t row_sum_word(int64_t rows_p, int64_t nkb, int n)
{
    return rows_p * nkb * n * (kKBlock / 32);
}

struct GemmArgs {
    int64_t M, N, K;
    int64_t nkb;          // roundup(K,512)/128
    int p, q;
    const uint32_t *a;    // packed activations (null when a_codes is given)
    const uint8_t *a_codes;  // small-M kernels only: M x K activation codes, packed by the kernel itself; else null
    const uint32_t *w;    // packed weights
    const int32_t *a_sum; // per activation row: sum of its codes over the padded K
    const int32_t *w_sum; // per weight row: the same
    int32_t *c_i32;       // may be null
    uint16_t *c_f16;      // may be null
    const uint16_t *w_scale;  // may be null
    const uint16_t *a_scale;  // may be null
};

// Several problems of one launch (decode kernels): workgroups wg_end[i-1] .. wg_end[i]-1 work on g[i].
constexpr int kMaxGroup = 8;
struct GroupArgs {
    int count;
    int chunk_kb[kMaxGroup];  // per problem: k blocks of activations held on chip at a time (a multiple of 32, or all)
    int wg_end[kMaxGroup];
    GemmArgs g[kMaxGroup];
};

}  // namespace apmm
