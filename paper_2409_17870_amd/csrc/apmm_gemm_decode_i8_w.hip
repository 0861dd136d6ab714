// int8 small-M kernels (apmm_gemm_decode_i8.h) on packed activations of up to 4 bits: wide weights, and 3- and 4-bit weights
// beyond the K that the fp4 kernels sum exactly.
#include "apmm_gemm_decode_i8.h"

namespace apmm {

namespace {
template <int FA>
hipError_t launch_q(const GroupArgs &ga, int tt, int rt, hipStream_t stream)
{
    const int q = ga.g[0].q;
    if constexpr (FA == i8::kFields) {
        if (q == 3) return i8::launch_decode_forms<FA, 3>(ga, tt, rt, stream);
        if (q == 4) return i8::launch_decode_forms<FA, 4>(ga, tt, rt, stream);
    }
    if (q == 8) return i8::launch_decode_forms<FA, i8::kBytes>(ga, tt, rt, stream);
    if (q >= 5) return i8::launch_decode_forms<FA, i8::kNibbles>(ga, tt, rt, stream);
    return hipErrorInvalidValue;
}
}  // namespace

hipError_t launch_decode_i8_narrow(const GroupArgs &ga, int tt, int rt, hipStream_t stream)
{
    switch (ga.g[0].p) {
    case 1: return launch_q<1>(ga, tt, rt, stream);
    case 2: return launch_q<2>(ga, tt, rt, stream);
    default: return launch_q<i8::kFields>(ga, tt, rt, stream);
    }
}

}  // namespace apmm
