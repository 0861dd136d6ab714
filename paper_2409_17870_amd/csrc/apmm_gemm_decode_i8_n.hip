// int8 small-M kernels (apmm_gemm_decode_i8.h) on packed activations of 5 .. 7 bits.
#include "apmm_gemm_decode_i8.h"

namespace apmm {
hipError_t launch_decode_i8_nibbles(const GroupArgs &ga, int tt, int rt, hipStream_t stream) { return i8::launch_decode_q<i8::kNibbles>(ga, tt, rt, stream); }
}  // namespace apmm
