// Pieces shared by the small-M kernels: workgroup shape, the problem descriptor of a launch, group descriptors.
#pragma once
#include "apmm_mfma_common.h"

namespace apmm {

constexpr int kDecodeWaves = 8;
constexpr int kDecodeThreads = 64 * kDecodeWaves;
constexpr int kRowsPerWg = 16;  // output channels per channel tile

struct DecodeProblem {
    const uint32_t *w;
    const void *a;          // packed activations, or codes (CODES)
    int64_t N, K, M;
    uint16_t *c_f16;
    int32_t *c_i32;
    const uint16_t *w_scale, *a_scale;
};

// problem of this workgroup and its index among the problem's workgroups
__device__ __forceinline__ int pick_problem(DecodeProblem &pr, uint32_t misc, const GroupArgs &ga)
{
    int block = (int)blockIdx.x;
    const int count = (int)((misc >> 12) & 0xffu);
    if (count > 1) {
        int idx = 0, first = 0;
#pragma unroll
        for (int i = 0; i + 1 < kMaxGroup; ++i) {  // one load for all ends (make_group: no end lies behind the last problem's)
            const int end = ga.wg_end[i];
            if (block >= end) {
                idx = i + 1;
                first = end;
            }
        }
        if (idx > 0) {
            const GemmArgs &g = ga.g[idx];
            pr.w = g.w;
            pr.a = g.a_codes ? static_cast<const void *>(g.a_codes) : static_cast<const void *>(g.a);
            pr.N = g.N; pr.K = g.K; pr.M = g.M;
            pr.c_f16 = g.c_f16; pr.c_i32 = g.c_i32;
            pr.w_scale = g.w_scale; pr.a_scale = g.a_scale;
            block -= first;
        }
    }
    return block;
}

struct __attribute__((packed, aligned(1))) Codes16 { uint32_t x, y, z, w; };  // 16 codes at any address

// Codes k .. k + 15 of a row from a load clamped to the row's last sixteen: `past` codes before position k are shifted out
// and the row is followed by ones.
__device__ __forceinline__ uint4 shift_past(uint4 v, int past)
{
    if (past <= 0) return v;
    if (past >= 16) return make_uint4(~0u, ~0u, ~0u, ~0u);
    if (past & 8) v = make_uint4(v.z, v.w, ~0u, ~0u);
    if (past & 4) v = make_uint4(v.y, v.z, v.w, ~0u);
    const int s = 8 * (past & 3);
    return make_uint4(__builtin_amdgcn_alignbit(v.y, v.x, s), __builtin_amdgcn_alignbit(v.z, v.y, s),
                      __builtin_amdgcn_alignbit(v.w, v.z, s), __builtin_amdgcn_alignbit(~0u, v.w, s));
}

// Builds the launch descriptor of `count` problems, `rows_per_wg` output channels per workgroup.
template <class PassKb>
inline bool make_group(const GemmArgs *gs, int count, int rows_per_wg, PassKb pass_kb, GroupArgs &ga)
{
    if (count < 1 || count > kMaxGroup) return false;
    int64_t end = 0;
    ga.count = count;
    for (int i = 0; i < kMaxGroup; ++i) {
        const GemmArgs &g = gs[i < count ? i : count - 1];
        if (i < count) end += (g.N + rows_per_wg - 1) / rows_per_wg;
        if (end > 0x7fffffffLL) return false;
        ga.wg_end[i] = (int)end;
        ga.g[i] = g;
        ga.chunk_kb[i] = (int)pass_kb(g);
        if (ga.chunk_kb[i] < 1) return false;
    }
    return true;
}

}  // namespace apmm
