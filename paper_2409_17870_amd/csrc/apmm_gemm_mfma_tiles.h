// Tile choice and width dispatch of the E2M1 MFMA GEMM (apmm_gemm_mfma_direct.h).  One translation
// unit per activation width instantiates the kernels, so that they compile in parallel.
#pragma once
#include "apmm_gemm_mfma_direct.h"
#include "apmm_gemm_mfma_lds.h"

namespace apmm {
namespace mfma {

// Switches for A/B measurements of the launch rule exist only in builds with -DAPMM_DEBUG_SWITCHES; the
// product build reads no environment variable.
inline const char *debug_switch(const char *name)
{
#ifdef APMM_DEBUG_SWITCHES
    return std::getenv(name);
#else
    (void)name;
    return nullptr;
#endif
}

// Tile choice.  Outputs of more than one round of the direct kernel's best tile go to the kernel that shares its operands through
// LDS (apmm_gemm_mfma_lds.h), 128 x 128 with two or three workgroups to a compute unit; so do nearly all with 3- and 4-bit
// activations.  Microseconds, direct against LDS, operands and outputs in rotation (M x N x K):
//   W4A4 1024 x 11008 x 4096 fp16 54 / 39, both outputs 68 / 39; 512 x 13824 x 5120 34.8 / 32.0; 4096 x 4096 x 4096 53 / 43
//   W2A4 700 x 8000 x 1000 fp16 11.9 / 9.9, 1024 x 11008 x 4096 35 / 28; W3A3 1000 x 5003 x 3001 both 29.7 / 26.0
//   W2A2 1024 x 11008 x 4096 28.1 / 23.9, both 40 / 27; 2048 x 11008 x 4096 both 67 / 54; 3000 x 8000 x 700 26.3 / 21.6
//   one round, W2A2, operands warm: 2048 x 4096 x 4096 (256 x 128) 17.2 / 17.6, 512 x 13824 x 5120 18.6 / 20.1, 2048 x 2048 x 2048 (128 x
//   128) 7.5 / 8.4: direct.
template <int P, int Q>
hipError_t launch_tiles(const GemmArgs &g, hipStream_t stream)
{
    const int64_t tiles128 = ((g.M + 127) / 128) * ((g.N + 127) / 128);
    static const char *forced = debug_switch("APMM_MFMA_TILE");
    static const char *no_split = debug_switch("APMM_MFMA_SPLIT");
    if constexpr (activation_field_form(P)) {
        (void)forced; (void)no_split;
        if constexpr (Q <= 2) {
            // One workgroup to a compute unit at most: the direct kernel's 128 x 128 tile (four wave tiles of 32 x 128, every
            // activation row block loaded by one wave) starts and ends faster, 1024 x 4096 x 512 / 1024 W2A4 5.8 / 7.2 against 6.1 /
            // 7.2 us, W1A4 5.4 / 6.2 against 5.7 / 6.7, and from K = 2048 on is slower: W2A4 0.80 - 0.99 of its time through LDS over six
            // outputs and K = 2048 - 8192, W1A4 0.82 - 1.04.  From K = 10240 on, where it has the outputs that the K split leaves, the
            // two are within 8 %.
            if (tiles128 <= 256 && (g.K < 2048 || g.K >= 10240)) return launch_direct_variant<P, Q, 1, 4>(g, stream);
            // With four tiles and more to a compute unit the 128 x 256 tile, two workgroups to a compute unit: fewer bytes from L2 and
            // LDS per product, longer runs per store.  W2A4 4096 x 4096 x 4096 39.4 -> 35.0 us, W1A4 35.3 -> 32.5; at three tiles equal
            // (1024 x 11008 x 4096 W2A4 30.0 / 29.1); below K = 2048 only with both outputs (4096 x 11008 x 1024 W2A4 81 -> 69 us, its
            // fp16 output alone 46 / 46, at K = 512 35 / 40).
            if (tiles128 > 3 * 256 && (g.K >= 2048 || (g.c_i32 && g.c_f16))) return launch_lds_variant<P, Q, 2, 4, 2>(g, stream);
        }
        return launch_lds_variant<P, Q, 2, 2, 2>(g, stream);
    } else {
        // Direct tiles: estimate each candidate as (rounds of 256 tiles) x (tile area) x (measured relative cost per MFMA of that tile
        // shape) and take the cheapest.  (Debug builds: APMM_MFMA_TILE=0..3 forces one.)
        struct Cand { int bm, bn; double cost; };
        // (4-bit weights: the words of four column blocks beside 256 accumulators would spill)
        const Cand cands[4] = {{256, 256, Q == 4 ? 1e9 : 1.0}, {256, 128, 1.2}, {128, 256, 1.2}, {128, 128, 1.2}};
        int best = 0;
        double best_t = 0;
        int64_t best_tiles = 0;
        const bool force = forced && forced[0] >= '0' && forced[0] <= '3' && !(Q == 4 && forced[0] == '0');
        if (force) best = forced[0] - '0';
        for (int c = 0; !force && c < 4; ++c) {
            const int64_t tiles = ((g.M + cands[c].bm - 1) / cands[c].bm) * ((g.N + cands[c].bn - 1) / cands[c].bn);
            const double t = (double)((tiles + 255) / 256) * cands[c].bm * cands[c].bn * cands[c].cost;
            if (c == 0 || t < best_t) {
                best = c;
                best_t = t;
                best_tiles = tiles;
            }
        }
        if (best_tiles > 256) return launch_lds_variant<P, Q, 2, 2, 3>(g, stream);
        switch (best) {
        case 0: {
            // Two-phase kernels (part of the store under the k loop).  APMM_MFMA_SPLIT=0, 2, 3 forces the one-phase,
            // the even or the uneven one where usable (debugging); otherwise the measured rule.  A split pays when
            // the store is exposed and the memory system is the limit: one round of tiles on most of the chip
            // (with more rounds the next tile's k loop already covers the store, with few tiles the store is
            // fast), K of at most 16 stages (beyond, the slower k loop costs what the store saves).
            // The uneven cut wins over the even one when the weight group is a single plane (cheapest expansion,
            // which the short second phase repeats per row block).
            const int64_t nst = g.nkb / 2;
            const int64_t tiles = ((g.M + 255) / 256) * ((g.N + 255) / 256);
            const bool pays = nst <= 16 && tiles > 128 && tiles <= 256;
            const char want = no_split ? no_split[0] : 0;
            if constexpr (Q == 1) {
                const bool ok3 = direct_split_usable<P, Q, 4, 4, 3>(g);
                if (ok3 && (want == '3' || (want == 0 && pays))) return launch_direct_variant<P, Q, 4, 4, 3>(g, stream);
            }
            if constexpr (Q <= 2) {
                const bool ok2 = direct_split_usable<P, Q, 4, 4, 2>(g);
                if (ok2 && (want == '2' || (want == 0 && pays))) return launch_direct_variant<P, Q, 4, 4, 2>(g, stream);
            }
            if constexpr (Q <= 3) return launch_direct_variant<P, Q, 4, 4>(g, stream);
            else return hipErrorInvalidValue;  // (never chosen)
        }
        case 1: return launch_direct_variant<P, Q, 4, 2>(g, stream);
        case 2: return launch_direct_variant<P, Q, 2, 4>(g, stream);
        default: return launch_direct_variant<P, Q, 2, 2>(g, stream);
        }
    }
}

template <int P>
hipError_t launch_fp4_p(const GemmArgs &g, hipStream_t stream)
{
    switch (g.q) {
    case 1: return launch_tiles<P, 1>(g, stream);
    case 2: return launch_tiles<P, 2>(g, stream);
    case 3: return launch_tiles<P, 3>(g, stream);
    case 4: return launch_tiles<P, 4>(g, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace mfma
}  // namespace apmm
