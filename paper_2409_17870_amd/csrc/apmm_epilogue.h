// Output stage shared by the GEMM kernels: the recovered int32 value is stored as is
// (the 32-bit output of paper Sec. 3.2) and/or scaled per token and per output channel
// in fp32 and rounded once to binary16.
#pragma once
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>
#include "apmm_layout.h"

namespace apmm {

__device__ __forceinline__ float half_bits_to_float(uint16_t bits)
{
    return __half2float(__ushort_as_half(bits));
}

__device__ __forceinline__ uint16_t float_to_half_bits(float x)
{
    return __half_as_ushort(__float2half_rn(x));
}

// fp16 results in pairs of columns: lane l holds column l of rows r (x0) and r + 1 (x1), and stores one dword, the even lane of a lane
// pair both columns of row r, the odd lane both of row r + 1.  half_pair rounds the two into one register (low, high half), swap_pair
// exchanges halves between the lanes: a lane permute and a byte permute, whose selector is the lane's for good.  Six operations a pair of results (two of
// them products with the token scales) where selects, masks and shifts took twelve, and that much less code for the K-split kernels to
// fetch at their end.  Launches inside a graph: W2A4 512 x 5120 x 5120 13.4 -> 13.2 us, 512 x 5120 x 13824 23.8 -> 23.6, W8A8 512 x 4096 x 4096 15.3 -> 15.2, 2048 x 11008 x 2048 66.1 ->
// 64.1; through LDS and in the direct tiles with a line's pieces stored together (apmm_gemm_mfma_lds.h), W2A2 1024 x 11008 x 4096 24.9 -> 24.6.  (By hand: left to itself the compiler makes four products and a conversion of two, which rounds once
// more than the single results' mixed multiplication.)  The direct tiles, but for the 256 x 256 ones, which spill with it: W2A2 2048 x 4096 x 2048 12.7 ->
// 12.2, 512 x 13824 x 5120 19.0 -> 18.5, W2A4 1024 x 4096 x 1024 8.1 -> 7.9, W1A4 1024 x 4096 x 512 5.6 -> 5.4.
__device__ __forceinline__ uint32_t half_pair(float x0, float x1, float y)
{
    uint32_t h;
    asm("v_fma_mixlo_f16 %0, %1, %2, 0" : "=v"(h) : "v"(x0), "v"(y));
    asm("v_fma_mixhi_f16 %0, %1, %2, 0" : "+v"(h) : "v"(x1), "v"(y));
    return h;
}
__device__ __forceinline__ uint32_t swap_pair_selector(bool odd) { return odd ? 0x03020706u : 0x05040100u; }
__device__ __forceinline__ uint32_t swap_pair(uint32_t mine, uint32_t selector)
{
    const uint32_t other = (uint32_t)__builtin_amdgcn_mov_dpp((int)mine, 0xB1, 0xf, 0xf, true);  // quad_perm [1, 0, 3, 2]
    return __builtin_amdgcn_perm(other, mine, selector);
}

// scale for row m / column n (1.0f when the vector is absent)
__device__ __forceinline__ float load_scale(const uint16_t *scale, int64_t idx)
{
    return scale ? half_bits_to_float(scale[idx]) : 1.0f;
}

// The same as raw binary16 bits, for kernels that request the scale long before they need it: the conversion
// is a use of the loaded value, and a use is where the wave waits for the load.
__device__ __forceinline__ uint32_t load_scale_bits(const uint16_t *scale, int64_t idx)
{
    return scale ? (uint32_t)scale[idx] : 0x3c00u;  // 1.0
}

// Pins the first use of a value loaded early to this point of the program: without it the compiler moves pure
// arithmetic on the value (a conversion, a multiply) up to the load, and the wave waits there for the load, and
// for every load issued before it.
__device__ __forceinline__ uint32_t use_here(uint32_t v)
{
    asm volatile("" : "+v"(v));
    return v;
}

// A copy in a register of its own: a lane permute that moves nothing, which the compiler does not see through.
__device__ __forceinline__ uint32_t copy_here(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xE4, 0xf, 0xf, true);  // quad_perm [0, 1, 2, 3]
}

// Before and behind a run of streaming stores: without them the compiler takes the run and the same run of plain stores on the other
// side of a branch for one, from either end, and drops the hint.
__device__ __forceinline__ void edge_of_streaming() { asm volatile("; streaming stores"); }

__device__ __forceinline__ void store_output(const GemmArgs &g, int64_t m, int64_t n, int32_t c, float sa,
                                             float sw)
{
    const int64_t o = m * g.N + n;
    if (g.c_i32) g.c_i32[o] = c;
    if (g.c_f16) g.c_f16[o] = float_to_half_bits((float)c * sa * sw);
}

}  // namespace apmm
