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
    // rounds of tiles times the time of one, in 10 ns (W8A8: a k block costs 0.33 us with K split, 0.94 us for four times
    // the outputs in the other arrangement; beginning, end and store about 4.5 us each)
    const int64_t small = ((g.M + 63) / 64) * ((g.N + 127) / 128), large = ((g.M + 127) / 128) * ((g.N + 255) / 256);
    const bool ksplit = (small + 255) / 256 * (33 * g.nkb + 450) <= (large + 255) / 256 * (94 * g.nkb + 450);
    if (g.p == 8) return launch_gemm_mfma_i8_b(g, stream, ksplit);
    if (g.p >= 5) return launch_gemm_mfma_i8_n(g, stream, ksplit);
    return launch_gemm_mfma_i8_w(g, stream, ksplit);
}

}  // namespace apmm
