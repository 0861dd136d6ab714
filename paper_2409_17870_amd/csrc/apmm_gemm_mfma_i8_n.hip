// int8 GEMM kernels (apmm_gemm_mfma_i8.h) for activations of 5 .. 7 bits and 1..8-bit weights.
#include "apmm_gemm_mfma_i8.h"

namespace apmm {

hipError_t launch_gemm_mfma_i8_n(const GemmArgs &g, hipStream_t stream, bool ksplit)
{
    switch (g.q) {
    case 1: return i8::launch_forms<i8::kNibbles, 1>(g, stream, ksplit);
    case 2: return i8::launch_forms<i8::kNibbles, 2>(g, stream, ksplit);
    case 3: return i8::launch_forms<i8::kNibbles, 3>(g, stream, ksplit);
    case 4: return i8::launch_forms<i8::kNibbles, 4>(g, stream, ksplit);
    case 8: return i8::launch_forms<i8::kNibbles, i8::kBytes>(g, stream, ksplit);
    default: return i8::launch_forms<i8::kNibbles, i8::kNibbles>(g, stream, ksplit);
    }
}

}  // namespace apmm
