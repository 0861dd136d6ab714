// int8 GEMM kernels (apmm_gemm_mfma_i8.h) for activations of up to 4 bits: wide weights, and 3- and 4-bit weights beyond
// the K that the fp4 kernels sum exactly.
#include "apmm_gemm_mfma_i8.h"

namespace apmm {

namespace {
template <int FA>
hipError_t launch_q(const GemmArgs &g, hipStream_t stream, bool ksplit)
{
    if constexpr (FA == i8::kFields) {
        if (g.q == 3) return i8::launch_forms<FA, 3>(g, stream, ksplit);
        if (g.q == 4) return i8::launch_forms<FA, 4>(g, stream, ksplit);
    }
    if (g.q == 8) return i8::launch_forms<FA, i8::kBytes>(g, stream, ksplit);
    if (g.q >= 5) return i8::launch_forms<FA, i8::kNibbles>(g, stream, ksplit);
    return hipErrorInvalidValue;
}
}  // namespace

hipError_t launch_gemm_mfma_i8_w(const GemmArgs &g, hipStream_t stream, bool ksplit)
{
    switch (g.p) {
    case 1: return launch_q<1>(g, stream, ksplit);
    case 2: return launch_q<2>(g, stream, ksplit);
    default: return launch_q<i8::kFields>(g, stream, ksplit);
    }
}

}  // namespace apmm
