// int8 matrix-unit GEMM (apmm_gemm_mfma_i8.h): coverage and launch rule.  The kernels are instantiated in
// apmm_gemm_mfma_i8_n.hip (activations of 5 .. 7 bits), _b.hip (8 bits) and _w.hip (up to 4 bits, mostly wide weights).
#include "apmm_kernels.h"

namespace apmm {

hipError_t launch_gemm_mfma_i8_n(const GemmArgs &g, hipStream_t stream, bool ksplit);
hipError_t launch_gemm_mfma_i8_b(const GemmArgs &g, hipStream_t stream, bool ksplit);
hipError_t launch_gemm_mfma_i8_w(const GemmArgs &g, hipStream_t stream, bool ksplit);

// Every pair of widths with a code of more than four bits, and activations of 3, 4 bits with weights of 3, 4 bits, whose
// fp4 kernels stop at K = 18432 (W4A4).
bool gemm_mfma_i8_supported(const GemmArgs &g)
{
    return (g.p > 4 || g.q > 4 || (g.p > 2 && g.q > 2)) && g.M <= 0x7fffffffLL && g.N <= 0x7fffffffLL && g.K <= 0x7fffffffLL;
}

hipError_t launch_gemm_mfma_i8(const GemmArgs &g, hipStream_t stream)
{
    // Rounds of tiles times the time of one, in 10 ns of W8A8 (a k block costs 0.33 us with K split, 0.94 us for four times
    // the outputs in the other arrangement; beginning, end and store about 4.5 us each).  Against that the tiles of the other
    // arrangement, whose waves form the bytes of every row twice, cost more where that takes most: weights in nibbles, and
    // folded ones under nibbles (W6A6 1024 x 4096 x 1024 24.3 against 19.6 us with K split, 512 x 11008 x 4096 63.0 against 57.2;
    // W3A6 and W5A8 likewise, while W8A8 takes 14.9 / 15.0 and 34.4 / 38.9 us there).  Over 19 outputs and 20 pairs of
    // widths the rule is within 6 % of the faster arrangement (24 % with the costs of W8A8 for all).
    const bool forming = nibble_form(g.q) || (weight_folded_form(g.q) && nibble_form(g.p)), folded = weight_folded_form(g.q);
    const int64_t per_kb = forming ? 128 : 94, ends = forming ? 900 : folded ? 700 : 450;
    const int64_t small = ((g.M + 63) / 64) * ((g.N + 127) / 128), large = ((g.M + 127) / 128) * ((g.N + 255) / 256);
    const bool ksplit = (small + 255) / 256 * (33 * g.nkb + 450) <= (large + 255) / 256 * (per_kb * g.nkb + ends);
    if (g.p == 8) return launch_gemm_mfma_i8_b(g, stream, ksplit);
    if (g.p >= 5) return launch_gemm_mfma_i8_n(g, stream, ksplit);
    return launch_gemm_mfma_i8_w(g, stream, ksplit);
}

}  // namespace apmm
