// Matrix-unit GEMM kernels whose four waves split K (apmm_gemm_mfma_ksplit.h): launch rule.  The kernels are
// instantiated in apmm_gemm_mfma_ksplit_p<P>.hip, one translation unit per activation width.
#include "apmm_kernels.h"

namespace apmm {

hipError_t launch_gemm_mfma_ksplit_p1(const GemmArgs &g, hipStream_t stream, int wn);
hipError_t launch_gemm_mfma_ksplit_p2(const GemmArgs &g, hipStream_t stream, int wn);
hipError_t launch_gemm_mfma_ksplit_p3(const GemmArgs &g, hipStream_t stream, int wn);
hipError_t launch_gemm_mfma_ksplit_p4(const GemmArgs &g, hipStream_t stream, int wn);

namespace {

// 128 x 256 tiles (32 below), one to a compute unit, for an fp16 output of 2-bit weights under 3- and 4-bit activations that has more than one
// round of 128 x 128: 160 bytes of operands per K for what two tiles of 128 x 128 take 256, in a longer start and end.  Time over that of the
// kernel with two 128 x 128 tiles to a compute unit, operands and outputs in rotation, W2A4: K = 4096 / 5120 / 8192 / 11008, 512 x 13824 0.85 / 0.80 / 0.79 /
// 0.74, 512 x 11008 1.03 / 0.82 / 0.78 / 0.75, 384 x 13824 0.92 / 0.84, 640 x 12288 0.91 / 0.86, 256 x 22016 0.87 / 0.82 / 0.78 / 0.74; at K = 6144 1024 x 5120 0.92,
// 1024 x 7680 0.86 - 0.91.  Up to 64 tokens the small-M kernel is the other one (33 and 64 tokens x 49160 - 65536, K = 4096 and 6144: 0.38 - 0.48); 65 - 128
// tokens from 33000 channels on 0.81 - 0.96 at K = 6144.  int32 alone 0.96 - 1.06, both outputs 1.00 - 1.17.  (Operands that fit the
// last-level cache: 512 x 13824 x 5120 1.02, 512 x 16384 x 4096 1.08.)
// Not where few compute units would have a second 128 x 128 tile: three rows of tiles and up to 264 tiles 1.07 / 1.04 / 1.05 / 1.04 / 1.02 at K = 4096 / 5120 /
// 6144 / 8192 / 11008 (384 x 11264).  At K = 6144 513 to 640 tokens 1.03 at 265 tiles and 0.97 at 280, 512 x 8448 and 8704 1.02 and 0.90 at 280, more tokens
// 1.04 - 1.06 at 258 - 264 tiles, 0.95 - 1.03 at 304, 0.92 - 1.0 at 320; from K = 6656 on 0.99 - 1.02 at 264.  At K = 4096 the other kernel's time is one of two by
// where its operands lie (512 x 11776 17.3 or 20.6 us, this one 18.5): over five placings each 1.10 at 257 x 11008 and 385 x 11008, 1.06 at 384 x 11776, 0.98
// at 384 x 12288, 0.95 at 320 x 14336; 1.12 at 257 x 17408; 512 x 10240 - 11776 0.98 - 1.05, 512 x 12288 0.95; 513 x 12288 1.05, 640 x 11520 1.04, 640 x
// 12288 0.90; 65 x 40000 1.04, 129 x 32768 0.98, 256 x 17408 0.89: the line lies at outputs of 4.4, 4.6 and 7.5 million.  Below: K = 3584 512 x 13824 1.03, 640 x 11008 1.10.
bool wide_tile_pays(const GemmArgs &g)
{
    if (!activation_field_form(g.p) || g.q != 2 || g.c_i32) return false;
    const int64_t rows = (g.M + 127) / 128, tiles128 = rows * ((g.N + 127) / 128), tiles256 = rows * ((g.N + 255) / 256);
    if (tiles128 <= 256 || tiles256 > 256 || (rows == 3 && tiles128 <= 264)) return false;
    if (g.nkb >= 52) return true;
    if (g.nkb >= 48 && tiles128 >= (g.M <= 640 ? 276 : 320)) return true;
    if (g.M > 640 || g.N < 10240) return false;
    return g.nkb >= 36 || (g.nkb == 32 && (g.M <= 64 || g.M * g.N >= (g.M <= 256 ? 4400000 : g.M <= 512 ? 4600000 : 7500000)));
}

// Tile width (column blocks of 32: 2, 4, 5 or 6; the tile has two row blocks): the one that fills most of the 256
// compute units in a single round of tiles, i.e. the narrowest with at most 256 tiles, or 0 when every width needs
// more than one round.  Activations in the group form (1 and 2 bits) have the 64 x 64 and 64 x 128 tiles only, weights of
// 3 and 4 bits no 64 x 192 tile (their words would not fit the registers).
int one_round_width(const GemmArgs &g)
{
    int best = 0;
    int64_t best_tiles = 0;
    for (int wn = 2; wn <= (!activation_field_form(g.p) ? 4 : g.q <= 2 ? 6 : 5); ++wn) {
        if (wn == 3) continue;
        const int64_t tiles = ((g.M + 63) / 64) * ((g.N + 32 * wn - 1) / (32 * wn));
        if (tiles <= 256 && tiles > best_tiles) {
            best = wn;
            best_tiles = tiles;
        }
    }
    if (best == 0 && wide_tile_pays(g)) return 32;
    // 128 x 128 tiles (16 here) where all narrower ones need a second round
    const int64_t tiles128 = ((g.M + 127) / 128) * ((g.N + 127) / 128);
    if (best == 0 && g.q >= 2 && g.nkb >= (g.q > 2 ? 32 : activation_field_form(g.p) ? 88 : 76) && tiles128 <= 256) return 16;
    return best;
}

}  // namespace

bool gemm_mfma_ksplit_supported(const GemmArgs &g) { return gemm_mfma_fp4_supported(g); }

// Launch rule, measured against the large-tile kernel inside a graph; with more than one round of tiles the large
// tiles win by 30 - 70 % (their fixed costs are paid once per larger tile), so one round is a condition throughout.
//   Field form (3, 4 bits; W2A4 and W1A4, 512 x 5120 outputs, fp16 output): slower below K = 4096 (the exchange
//   through LDS and the colder start of waves that each begin at another place of K cost about 2 us per tile),
//   equal to 10 % faster at K = 5120 (14.2 against 14.5 us on one box, 12.1 against 13.4 us on another), 15 - 26 %
//   faster at K = 13824 (28.2 against 33.1, 22.5 against 30.4 us): the k loop gains 0.5 us per 1024 elements of K.
//   Taken from K = 5120 on; with the 64 x 128 tile (outputs of up to 256 of them, e.g. up to 512 tokens at 4096
//   channels or 128 at 11008) already from K = 3072 on: 1 - 256 tokens at 4096 x 4096 9.4 - 9.8 against 11.2 - 12.6 us,
//   at 4096 x 11008 15.5 - 16.2 against 22.7 - 24.1 us, equal at K = 1024.
//   Group form (1, 2 bits; W2A2 and W1A2, fp16 or int32 output), where the large-tile kernel has 128 x 128 tiles for
//   these outputs: 512 x 4096 outputs 5.9 / 7.3 / 9.9 / 16.6 us against 6.7 / 7.5 / 8.6 / 11.6 us here at K = 1024 / 2048 /
//   4096 / 8192; 512 x 4096 x 11008 22.0 against 13.8 us; 65 x 4096 and 96 x 11008 outputs faster at every K (10.7
//   against 7.9 us at K = 4096).  Taken from K = 3072 on, and at every K up to 128 tokens.
//   The 128 x 128 tile (1024 x 4096 outputs and the like, every width; large tiles against this, K = 2048 / 4096 / 8192 /
//   11008): W4A4 12.1 / 19.1 / 34.6 / 45.3 against 13.2 / 16.8 / 25.7 / 32.3 us, W3A3 11.2 / 16.6 / 29.9 / 41.0 against 12.8 /
//   16.2 / 24.5 / 30.7, W4A2 9.7 / 15.5 / 27.0 / 34.4 against 11.6 / 14.6 / 21.9 / 26.5: taken from K = 4096 on with weights of 3
//   and 4 bits.  (This and the next sentence: the register form of the tile against the direct tiles.)  2 bits: this over the large tiles, 512 x 6144 / 640 x 5120 / 768 x 4096 / 512 x 8192 / 1024 x 4096 outputs, W2A1
//   1.07 / 1.05 / 1.05 / 1.04 / 1.06 at K = 8192, 0.99 - 1.02 at 9216, 0.98 - 1.03 at 9728, 0.94 - 0.99 at 11264; W2A2 1.01 -
//   1.04, 0.96 - 1.02, 0.96 - 1.03, 0.92 - 0.99; W2A4 (the last three) 1.10, 1.04, 1.03 - 1.05 and 1.00 - 1.01: taken from K =
//   9728 on, with 3- and 4-bit activations from 11264 on (13824: 0.96 - 1.00).  W1A4 26.4 against 28.8 us at K = 11008: not
//   taken with 1 bit.
//   The form through LDS that serves K up to about 9216 and 2-bit weights now, over the large tiles of now (1024 x 4096 / 3072,
//   2048 x 2048, 640 x 6144, 700 x 5000, one or both outputs, operands and outputs in rotation): W3A1 and W3A2 1.02 - 1.21 at
//   K = 512, 0.95 - 1.08 at 2048, 0.96 - 1.10 at 3072 and 3584; W3A4 0.97 - 1.16, 0.94 - 1.07, 0.89 - 1.02; W4A2 0.98 - 1.15,
//   0.89 - 1.04, 0.86 - 1.07; W4A4 1.01 - 1.18, 1.03 - 1.22, 0.92 - 1.04; W2A1 and W2A2 1.02 - 1.22 at 1024, 0.94 - 1.14 at 2048,
//   0.95 - 1.10 at 4096, 0.91 - 1.06 at 6144 - 9216; W2A4 0.98 - 1.10 at 1024, 0.96 - 1.10 at 2048, 0.93 - 1.01 at 4096,
//   0.86 - 1.04 at 6144 - 9216, 0.82 - 1.04 at 10240 and 10752.  The lines are on the safe side; the one of W2A4 could lie at
//   6144, that of W3A4 and W4A4 at 3584.
//   The 64 x 64 tile (outputs of up to 256 of them: up to 256 tokens at 4096 channels, 128 at 8192), with weights of 1 and
//   2 bits: 65 - 256 tokens at 4096 x 4096 5.3 - 5.9 us (W1A1, W2A2), 6.9 - 7.4 us (W2A4) against 7.5 - 8.5 and 9.6 - 9.9 us with
//   the 64 x 128 tile and 9.3 - 11.5 us on the large tiles; at 4096 x 11008 7.4 - 8.5 and 10.7 - 11.9 against 11.0 - 12.1 and
//   15.8 - 16.5 us; at K = 1024 4.4 - 5.0 against 5.5 - 6.6 us on the large tiles.  With 3 and 4 bits 6.8 - 7.4 us (W3A3) and
//   6.7 - 7.5 us (W4A4) at 4096 x 4096, 11.5 - 12.9 and 11.7 - 13.4 us at 4096 x 11008 against 14 - 18 and 31 - 34 us on the
//   large tiles.  Taken at every K.
bool gemm_mfma_ksplit_pays(const GemmArgs &g)
{
    if (!gemm_mfma_ksplit_supported(g) || one_round_width(g) == 0) return false;
    const int width = one_round_width(g);
    if (width == 2 || width >= 16) return true;
    if (activation_field_form(g.p)) return g.nkb >= 40 || (width == 4 && g.nkb >= 24);
    return g.nkb >= 24 || g.M <= 128;
}

hipError_t launch_gemm_mfma_ksplit(const GemmArgs &g, hipStream_t stream)
{
    int wn = one_round_width(g);
    if (wn == 0) wn = activation_field_form(g.p) ? 5 : 4;  // explicit request for a shape of several rounds
    switch (g.p) {
    case 1: return launch_gemm_mfma_ksplit_p1(g, stream, wn);
    case 2: return launch_gemm_mfma_ksplit_p2(g, stream, wn);
    case 3: return launch_gemm_mfma_ksplit_p3(g, stream, wn);
    case 4: return launch_gemm_mfma_ksplit_p4(g, stream, wn);
    }
    return hipErrorInvalidValue;
}

}  // namespace apmm
