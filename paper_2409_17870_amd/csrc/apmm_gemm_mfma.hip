// Dispatch of the MFMA GEMMs (design A).  The kernels are instantiated in apmm_gemm_mfma_p<P>.hip,
// one translation unit per activation width, so that they compile in parallel.
#include <cstdio>

#include "apmm_kernels.h"

namespace apmm {

namespace {
thread_local KernelTiming g_timing = {nullptr, nullptr};
// The name of the last kernel as its format and arguments: written out when it is asked for, since a product's call is not much longer than
// its launch (16 x 256 x 512 from Python 5.1 -> 4.7 us, with a shorter binding, the two in turn in one process).
struct KernelName {
    const char *fmt = "";
    KernelNameArg arg[kMaxKernelNameArgs];
    int count = 0;
    char written[96];
};
thread_local KernelName g_last_kernel;
}
void keep_kernel_name(const char *fmt, const KernelNameArg *args, int count)
{
    KernelName &k = g_last_kernel;
    k.fmt = fmt;
    k.count = count;
    for (int i = 0; i < count; ++i) k.arg[i] = args[i];
}
const char *last_kernel()
{
    KernelName &k = g_last_kernel;
    size_t at = 0;
    int n = 0;
    for (const char *c = k.fmt; *c && at < sizeof(k.written) - 1; ++c) {
        if (*c != '%') {
            k.written[at++] = *c;
            continue;
        }
        if (c[1]) ++c;
        if (n == k.count) continue;
        const KernelNameArg &a = k.arg[n++];
        const size_t room = sizeof(k.written) - at;
        const size_t w = (size_t)(a.text ? std::snprintf(k.written + at, room, "%s", a.text) : std::snprintf(k.written + at, room, "%d", a.number));
        at += w < room ? w : room - 1;
    }
    k.written[at] = 0;
    return k.written;
}
void set_kernel_timing(hipEvent_t start, hipEvent_t stop) { g_timing = KernelTiming{start, stop}; }
KernelTiming take_kernel_timing()
{
    const KernelTiming t = g_timing;
    g_timing = KernelTiming{nullptr, nullptr};
    return t;
}

hipError_t launch_gemm_mfma_fp4_p1(const GemmArgs &g, hipStream_t stream);
hipError_t launch_gemm_mfma_fp4_p2(const GemmArgs &g, hipStream_t stream);
hipError_t launch_gemm_mfma_fp4_p3(const GemmArgs &g, hipStream_t stream);
hipError_t launch_gemm_mfma_fp4_p4(const GemmArgs &g, hipStream_t stream);

// The fp32 accumulator runs from the recovery terms to C through integer partial sums; all of them are
// below 4 K' (2^p - 1)(2^q - 1) in magnitude, which must stay below 2^24 for the sums to be exact.
bool gemm_mfma_fp4_supported(const GemmArgs &g)
{
    if (g.p < 1 || g.p > 4 || g.q < 1 || g.q > 4) return false;
    const int64_t unit = (int64_t)((1 << g.p) - 1) * ((1 << g.q) - 1);
    return 4 * g.nkb * kKBlock * unit < (1 << 24);
}

hipError_t launch_gemm_mfma_fp4(const GemmArgs &g, hipStream_t stream)
{
    switch (g.p) {
    case 1: return launch_gemm_mfma_fp4_p1(g, stream);
    case 2: return launch_gemm_mfma_fp4_p2(g, stream);
    case 3: return launch_gemm_mfma_fp4_p3(g, stream);
    case 4: return launch_gemm_mfma_fp4_p4(g, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace apmm
