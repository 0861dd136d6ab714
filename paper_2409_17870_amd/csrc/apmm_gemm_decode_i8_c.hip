// int8 small-M kernels (apmm_gemm_decode_i8.h) on unpacked activation codes.
#include "apmm_gemm_decode_i8.h"

namespace apmm {
hipError_t launch_decode_i8_codes(const GroupArgs &ga, int tt, int rt, hipStream_t stream) { return i8::launch_decode_q<i8::kCodes>(ga, tt, rt, stream); }
}  // namespace apmm
