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

// Tile choice.  Most outputs of more than one round of the direct kernel's best tile go to the kernel that shares its operands through
// LDS (apmm_gemm_mfma_lds.h), 128 x 128 with two or three workgroups to a compute unit; so do nearly all with 3- and 4-bit
// activations.  Microseconds, direct against LDS, operands and outputs in rotation (M x N x K):
//   W4A4 1024 x 11008 x 4096 fp16 54 / 39, both outputs 68 / 39; 512 x 13824 x 5120 34.8 / 32.0; 4096 x 4096 x 4096 53 / 43
//   W2A4 700 x 8000 x 1000 fp16 11.9 / 9.9, 1024 x 11008 x 4096 35 / 28; W3A3 1000 x 5003 x 3001 both 29.7 / 26.0
//   W2A2 1024 x 11008 x 4096 28.1 / 23.9, both 40 / 27; 2048 x 11008 x 4096 both 67 / 54; 3000 x 8000 x 700 26.3 / 21.6
//   one round, W2A2, operands warm: 2048 x 4096 x 4096 (256 x 128) 17.2 / 17.6, 512 x 13824 x 5120 18.6 / 20.1, 2048 x 2048 x 2048 (128 x
//   128) 7.5 / 8.4: direct.
inline int64_t tile_count(const GemmArgs &g, int bm, int bn) { return ((g.M + bm - 1) / bm) * ((g.N + bn - 1) / bn); }

// 3- and 4-bit activations, whose direct tiles are 128 x 128 and, with 3-bit weights, 128 x 256: the shape (wave rows, wave columns) of
// those that are taken, 0 for the kernel through LDS.  Figures: time through LDS over that of the direct tile, operands and outputs in
// rotation.
struct DirectTile { int wm, wn; };
template <int P, int Q>
inline DirectTile field_direct_tile(const GemmArgs &g)
{
    const int64_t tiles = tile_count(g, 128, 128), tiles256 = tile_count(g, 128, 256);
    const bool i32_alone = !g.c_f16, f16_alone = !g.c_i32;
    const bool some = tiles >= 64;  // (fewer go to the K split unless these kernels are asked for by id)
    if (Q <= 2 && tiles <= 256) {
        // One workgroup to a compute unit at most: four wave tiles of 32 x 128, every activation row block loaded by one wave, start
        // and end faster, 1024 x 4096 x 512 / 1024 W2A4 5.8 / 7.2 against 6.1 / 7.2 us, W1A4 5.4 / 6.2 against 5.7 / 6.7.  From K = 10240 on
        // (1024 x 4096 / 3072, 2048 x 2048, 640 x 6144, 700 x 5000; up to K = 16384 with single bits) through LDS it would be 0.97 - 1.02 of
        // this for W1A3 and W1A4 int32 alone, 0.94 - 1.03 with fp16; for W2A4, below the 11264 of the K split, 0.90 - 1.00.
        if (g.K < 2048 || g.K >= 10240) return {1, 4};
        // Between, with single bits: int32 alone 1.00 - 1.17 (K = 2048: 1024 x 2048 1.14, 2048 x 2048 1.12; 6144: 0.99 - 1.05), fp16 alone up to 192 tiles
        // 1.01 - 1.05 at 2048, 0.95 - 1.06 at 2560, 0.94 - 1.01 at 3072; both outputs 0.79 - 0.97 but for the fewest tiles (512 x 3000, 96 of them, 1.03 -
        // 1.06).
        if (Q == 1 && some && (i32_alone || (g.K < 3072 && tiles <= (f16_alone ? 192 : 96)))) return {1, 4};
        // With two bits: int32 alone up to 128 tiles 1.03 - 1.05 at 2048, 0.99 - 1.03 at 2560; else 0.84 - 1.02.
        if (Q == 2 && some && i32_alone && g.K < 3072 && tiles <= 128) return {1, 4};
    }
    if (Q == 3) {
        // int32 alone: 512 x 4096, 256 x 8192, 640 x 6144, 512 x 5120 1.02 - 1.08 up to K = 512; at 1024 1.02 - 1.07 up to 160 tiles, 0.92 - 0.97 from 192 on
        if (some && i32_alone && tiles <= 256 && (g.K <= 512 || (g.K <= 1024 && tiles <= 160))) return {2, 2};
        // one full round of 128 x 256 tiles, 2048 x 4096, 2048 x 3584, 1792 x 4096, one output: 1.02 - 1.07 at K = 8192 and 11008, 0.98 - 1.03 at 6144
        if (!(g.c_i32 && g.c_f16) && g.K >= 8192 && tiles256 <= 256 && tiles256 >= 224) return {2, 4};
    }
    return {0, 0};
}

// 1- and 2-bit activations, more than one round (256) of the direct tile bm x bn that the cost model picks: where this tile still beats
// the kernel through LDS.  Figures as above.
template <int P, int Q>
inline bool rounds_go_direct(const GemmArgs &g, int bm, int bn, int64_t tiles)
{
    const int64_t rounds = (tiles + 255) / 256;
    const bool one = !(g.c_i32 && g.c_f16), full = tiles * 20 >= rounds * 256 * 19, nearly = tiles * 9 >= rounds * 256 * 8;
    // two full rounds of 256 x 256, fp16 alone, next to no sum: 4096 x 8192 W1A1 / W2A1 / W2A2 1.04 - 1.07
    if (Q <= 2 && rounds == 2 && full && !g.c_i32 && g.K <= 512 && bm == 256 && bn == 256) return true;
    if (Q == 3) {
        // 256 x 256, full rounds: 4096 x 8192, 8192 x 8192, 2048 x 16384 one output 1.00 - 1.11 at K = 4096, 1.05 - 1.17 at 6144, 1.09 - 1.20 beyond, both 1.04 - 1.13
        // from 8192 on; 8/9 of the rounds full (4096 x 11008) one output 1.05 - 1.08 at 8192
        if (bm == 256 && bn == 256) return full ? g.K >= (one ? 4096 : 8192) : nearly && one && g.K >= 8192;
        // 256 x 128: 2048 x 11008, 3000 x 8000 one output 1.00 - 1.06 at 8192, 1.02 - 1.08 at 11008
        return bm == 256 && nearly && one && g.K >= 8192;
    }
    if (Q == 4 && bm == 256) {
        // 256 x 128, two full rounds: 4096 x 4096, 2048 x 8192, 1024 x 16384 one output 1.00 - 1.07 at 6144, 1.02 - 1.13 beyond; both and more rounds up to 1.14
        // at 11008 (2048 x 16384, 1024 x 16384; 4096 x 8192 0.92 - 1.03)
        return full && rounds == 2 && g.K >= (one ? 6144 : 10240);
    }
    if (Q == 4 && P == 1) {
        // 128 x 128 with two workgroups through LDS on most compute units and three on some: 540 tiles (600 x 13824) 1.03 - 1.10 from K = 4096 on, 516
        // (320 x 22016, 700 x 11008) 1.00 - 1.11 up to 8192, 0.88 - 0.99 at 11008
        return tiles <= 576 && g.K >= 4096 && (tiles > 528 || g.K < 9728);
    }
    // 256 x 256, 2-bit codes on a side: 4096 x 8192, 2048 x 16384 fp16 alone 1.04 - 1.05 at 8192, 1.04 - 1.08 at 11008, int32 alone 1.03 - 1.05 at 11008
    return P + Q >= 3 && bm == 256 && bn == 256 && full && one && g.K >= (g.c_i32 ? 10240 : 8192);
}

template <int P, int Q>
hipError_t launch_tiles(const GemmArgs &g, hipStream_t stream)
{
    static const char *forced = debug_switch("APMM_MFMA_TILE");
    static const char *no_split = debug_switch("APMM_MFMA_SPLIT");
    if constexpr (activation_field_form(P)) {
        (void)forced; (void)no_split;
        const DirectTile direct = field_direct_tile<P, Q>(g);
        if constexpr (Q == 3) {
            if (direct.wm == 2) return direct.wn == 2 ? launch_direct_variant<P, Q, 2, 2>(g, stream) : launch_direct_variant<P, Q, 2, 4>(g, stream);
        }
        if constexpr (Q <= 2) {
            if (direct.wm == 1) return launch_direct_variant<P, Q, 1, 4>(g, stream);
            // With four tiles and more to a compute unit the 128 x 256 tile, two workgroups to a compute unit: fewer bytes from L2 and
            // LDS per product, longer runs per store.  W2A4 4096 x 4096 x 4096 39.4 -> 35.0 us, W1A4 35.3 -> 32.5; at three tiles equal
            // (1024 x 11008 x 4096 W2A4 30.0 / 29.1); below K = 2048 only with both outputs (4096 x 11008 x 1024 W2A4 81 -> 69 us, its
            // fp16 output alone 46 / 46, at K = 512 35 / 40).
            // With little more than a round of them (512) half of the second would be idle: 1500 x 11008, 516 tiles, and 4096 x 4128, 544, 128 x 128
            // over 128 x 256 0.87 - 0.95.
            const int64_t wide = tile_count(g, 128, 256), slots = (wide + 511) / 512 * 512;
            if (tile_count(g, 128, 128) > 3 * 256 && wide * 10 >= slots * 6 && (g.K >= 2048 || (g.c_i32 && g.c_f16))) return launch_lds_variant<P, Q, 2, 4, 2>(g, stream);
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
            const int64_t tiles = tile_count(g, cands[c].bm, cands[c].bn);
            const double t = (double)((tiles + 255) / 256) * cands[c].bm * cands[c].bn * cands[c].cost;
            if (c == 0 || t < best_t) {
                best = c;
                best_t = t;
                best_tiles = tiles;
            }
        }
        if (best_tiles > 256 && !rounds_go_direct<P, Q>(g, cands[best].bm, cands[best].bn, best_tiles)) return launch_lds_variant<P, Q, 2, 2, 3>(g, stream);
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
            const int64_t tiles = tile_count(g, 256, 256);
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
