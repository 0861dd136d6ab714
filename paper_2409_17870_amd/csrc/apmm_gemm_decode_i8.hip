// int8 small-M kernels (apmm_gemm_decode_i8.h): coverage and launch rule.  The kernels are instantiated in
// apmm_gemm_decode_i8_c.hip (unpacked activation codes), _b.hip (8 bits), _n.hip (5 .. 7 bits) and _w.hip (up to 4 bits).
#include "apmm_decode_common.h"

namespace apmm {

hipError_t launch_decode_i8_codes(const GroupArgs &ga, int tt, int rt, hipStream_t stream);
hipError_t launch_decode_i8_bytes(const GroupArgs &ga, int tt, int rt, hipStream_t stream);
hipError_t launch_decode_i8_nibbles(const GroupArgs &ga, int tt, int rt, hipStream_t stream);
hipError_t launch_decode_i8_narrow(const GroupArgs &ga, int tt, int rt, hipStream_t stream);

// The widths of the large int8 kernels, up to 64 tokens; unpacked codes in rows of at least one 16-byte load.
// Against the 64 x 128 tiles of the large kernels, W4A8 / W8A8 / W2A6: 64 x 4096 x 4096 6.3 / 8.3 / 8.8 us here, 11.4 / 18.7 /
// 12.4 us there; 64 x 4096 x 11008 14.2 / 17.8 / 17.9 against 26.7 / 42.4 / 24.5 us; but 64 x 11008 x 4096, where every one of
// 688 workgroups reads all the tokens, 16.4 / 19.9 / 24.5 against 13.7 / 20.7 / 13.1 us (32 tokens: 10.5 / 13.7 / 10.8
// against 12.7 / 19.9 / 13.1 us), hence the bound on the channels.
bool gemm_decode_i8_supported(const GemmArgs &g)
{
    return g.M >= 1 && (g.M <= 32 || (g.M <= 64 && g.N <= 8192)) && gemm_mfma_i8_supported(g) && (!g.a_codes || g.K >= 16);
}

hipError_t launch_gemm_decode_i8(const GemmArgs *gs, int count, int tt, hipStream_t stream)
{
    int64_t rows = 0;
    for (int i = 0; i < count; ++i) rows += gs[i].N;
    // two channel tiles per workgroup once single ones would need a second round of workgroups, two to a CU (11008 x 4096, 8
    // tokens from codes, W4A8 9.2 -> 8.4 us, W2A6 8.2 -> 6.5 us; at 4096 channels 4.8 -> 5.3 us, so not there); four token
    // tiles leave no registers for it
    const int rt = tt < 4 && rows > 2 * 256 * kRowsPerWg ? 2 : 1;
    GroupArgs ga;
    if (!make_group(gs, count, kRowsPerWg * rt, [](const GemmArgs &g) { return g.nkb; }, ga)) return hipErrorInvalidValue;
    if (gs[0].a_codes) return launch_decode_i8_codes(ga, tt, rt, stream);
    if (gs[0].p == 8) return launch_decode_i8_bytes(ga, tt, rt, stream);
    if (gs[0].p >= 5) return launch_decode_i8_nibbles(ga, tt, rt, stream);
    return launch_decode_i8_narrow(ga, tt, rt, stream);
}

}  // namespace apmm
