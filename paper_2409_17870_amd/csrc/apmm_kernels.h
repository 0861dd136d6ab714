// Host-side launchers of the library's kernels (internal; the public ABI is include/apmm.h).
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "apmm_layout.h"

namespace apmm {

constexpr int64_t kMostWorkItems = 0xffffffffLL;  // of one dimension of a launch

// Paper Sec. 4.1: decomposition into planes, reassembly into 32-bit words, concatenation.
// `field`: the field form of 3- and 4-bit activations instead of the group form (apmm_layout.h).
hipError_t launch_pack(const uint8_t *codes, int64_t rows, int64_t K, int bits, bool field, uint32_t *packed,
                       hipStream_t stream);
// Its rule for many rows: eight rows to a workgroup, code sums on the way, against a wave per packed tile and waves of their own for the sums (1 and 2
// bits: against a wave per row).  Time of eights over the other's, least and most of three settings: the same codes again and again, several states in the
// last-level cache, codes and output from and to memory.  What decides is how evenly its workgroups, all alike, fill the 256 compute units: `full`, the share of the
// last round of 256 that is there.
// 3 to 8 bits, K up to 4096 (a piece of 512 codes or none for each of eight waves): from 6144 rows on 0.34 - 0.96, of which fewer than 512 codes a row 0.34 - 0.91; 3072
// to 6143 rows, 0.8 full, 0.70 - 1.03 from 10 million codes on (7 million 0.85 - 1.05; 0.7 to 0.75 full 0.80 - 1.07); one round, 1700 rows and K = 3300 at least, 0.57 - 0.99 (1500 x
// 3072 0.90 - 1.03, 2048 x 3001 0.83 - 1.07); little more than one, 2100 to 2800 x 4096, 0.85 - 1.07.
// Longer rows: 0.95 full in one or two rounds, 0.88 in more, 0.63 - 1.05 (2048 x 5120 0.86 - 0.97, 2048 x 11008 0.69 - 0.77, from memory 0.99 - 1.05; 4096 x 8192 0.67 - 0.97, 5504 x 8192
// 0.75 - 0.96, 11008 x 11008 0.69 - 1.01); else from memory up to 1.08 (3600 and 6400 x 11008), 1.14 (4200 x 11008) and 1.35 (2100 x 11008).  Six slots and more, K beyond 7000, operand and output beyond the last-level cache: 4096 x 11008 0.95 - 1.02, 11008 x 11008 1.03 - 1.05.
// Two bits: from 45 million codes on, 0.88 full, 0.67 - 1.01 (8192 x 8192, the same codes again, 1.05; fewer codes 0.71 - 1.03; 2500 rows 0.84 - 1.27).  One bit: from 100 million
// on 0.71 - 0.91, the same codes again 0.91 - 1.06 (2500 rows 1.06 - 1.32).  Not where its launch would pass 2^32 work items, which the other's grid of three dimensions does not.
constexpr int kEightWaves = 8;  // most waves of pack_eights_kernel
inline int64_t pack_eights_threads(int64_t K) { return 64 * (K <= kEightWaves * kKPad ? round_up(K, kKPad) / kKPad : kEightWaves); }  // of eight rows
inline bool pack_by_eights(int64_t rows, int64_t K, int bits, bool field)
{
    const int64_t codes = rows * K, groups = round_up(rows, kRowBlock) / 8, rounds = (groups + 255) / 256;
    if (groups * pack_eights_threads(K) > kMostWorkItems) return false;
    auto full = [&](int percent) { return groups * 100 >= rounds * 256 * percent; };
    if (!field && bits <= 2) return rows >= 2048 && full(88) && codes >= (bits == 2 ? 45000000 : 100000000);
    if (K <= 4096) {
        if (rows >= 6144) return codes >= 4500000;
        return rows >= 3072 ? full(80) && codes >= 10000000 : rows >= 1700 && rows <= 2048 && K >= 3300;
    }
    const int slots = field ? 6 : bits;
    return rows >= 1700 && full(rounds <= 2 ? 95 : 88) && !(slots >= 6 && K > 7000 && codes > 40000000);
}
// Paper Sec. 3.1 + 4.1: per-row symmetric quantisation of binary16 features fused with the packing.
hipError_t launch_quantize_pack(const uint16_t *x, int64_t rows, int64_t K, int bits, bool field, uint32_t *packed,
                                uint16_t *scale, hipStream_t stream);
// Its rule for many rows in the field form: four rows to a workgroup of 128 lanes each, up to four groups of 32 elements to a lane.  Old / new,
// microseconds: 640 x 4096 5.2 / 4.6, 1024 x 4096 6.0 / 5.1, 1024 x 11008 13.1 / 10.1, 4096 x 2048 9.5 / 7.6, 4096 x 11008 48.5 / 28.7; on the other
// side 512 x 5120 4.8 / 5.8, 512 x 13824 8.9 / 9.4, 1024 x 2048 4.1 / 4.4, 4096 x 1500 9.8 / 10.5, 16 x 5120 3.2 / 4.9.
constexpr int kQuantLanes = 128;
inline int64_t quantize_groups(int64_t K) { return round_up(K, kKPad) / 32; }
inline int64_t quantize_lane_groups(int64_t K) { return (quantize_groups(K) + kQuantLanes - 1) / kQuantLanes; }
inline bool quantize_rows_by_four(int64_t rows, int64_t K)
{
    const int64_t lane_groups = quantize_lane_groups(K);
    if (rows <= 512 || K < 2048 || rows * K < 2500000 || lane_groups > 4) return false;
    // A few more workgroups than compute units and rows that the other kernel gives two waves, 2049 to 2560: new over old 1.04 - 1.10 at
    // 1100 to 1500 rows, 0.94 at 1024, 0.93 - 0.97 at 1600; one wave (2048) 0.88 - 0.92.
    if (lane_groups == 1) return !(K > 2048 && K <= 2560 && rows > 1024 && rows < 1600);
    // Where most lanes lack the last group (K = 4300: 144 groups on 128 lanes) it takes more rows: 513 x 4900 5.6 / 6.7, 641 x 4300 5.3 / 6.4, 577 x 5120
    // 5.6 / 6.2, 513 x 8704 7.0 / 7.8.  With a share f of the groups there, new over old is 1.00 - 1.05 at rows f from 440 to 480 and two
    // groups to a lane, 0.92 - 1.00 with three and four; 0.92 - 1.02 at 500 to 540.
    return rows * quantize_groups(K) >= (lane_groups == 2 ? 500 : 450) * lane_groups * kQuantLanes;
}
// Waves of a row in the kernel of one row to some waves: a group of 32 elements for every lane, as far as the row goes.  Beyond 8192 elements, time with eight over
// with four, least and most of three settings (the same features again and again, several states, from memory).  Up to 256 rows 0.75 - 1.01 (16 x 13824 four bits 4.11 -> 3.81 us,
// 16 x 11008 two bits 4.16 -> 3.65).  Whole k blocks: the field form, 300 to 512 rows, 0.91 - 1.00; the others, 300 to 1500 rows up to K = 16384, 0.91 - 1.11 (eight bits 800 x 13824 from
// memory 1.15): four; 2048 rows and more 0.91 - 0.99 where most lanes have a group (10752 and beyond), 1.02 - 1.24 where they have not (8704).  Rows that end inside a k
// block take the kernel with more registers, of which a compute unit holds three workgroups: 768 rows are one round.  Up to there 0.81 - 0.99, with 800 rows and more 1.00 - 1.09
// at two and five bits, 1.03 - 1.21 at eight; beyond 16384 0.92 - 1.16 at 800 to 1024 rows up to K = 22001 (four and eight bits above 1), 0.76 - 1.04 with more rows or longer
// ones.  Whole k blocks beyond 16384, 300 rows and more 0.80 - 1.03 (800 x 20480 from memory 0.90 - 1.11).  There sixteen over four up to 256 rows 0.56 - 0.96; over eight up to 100 rows 0.85 - 0.99,
// 512 and 1024 rows 0.93 - 1.4.
inline int quantize_waves(int64_t rows, int64_t K, bool field)
{
    const int64_t nkb = round_up(K, kKPad) / kKBlock;
    if (nkb <= 64) return nkb <= 16 ? 1 : nkb <= 32 ? 2 : 4;
    if (nkb > 128 && rows <= 256) return 16;
    if (round_up(rows, 64) * 512 > kMostWorkItems) return 4;  // 8 388 545 rows and more
    const bool ragged = K % kKBlock != 0;
    if (ragged) return (rows > 768 && nkb <= (rows <= 1024 ? 176 : 128)) ? 4 : 8;
    if (!field && nkb <= 128 && rows > 256 && rows < 2048) return 4;
    return nkb < 84 && rows > 1024 ? 4 : 8;
}
// Five workgroups to a compute unit instead of the seven or eight that its registers leave room for, in the kernel of one row to up to four waves,
// from 17 MB of packed output on: its stores are pieces of lines that other waves complete, and more rows under way push them out of L2 before.
// Eight over five, eight bits 4096 x 4608 / 4096 x 5632 / 4096 x 8192 / 4096 x 9216 / 3000 x 10240 0.97 / 1.08 / 1.12 / 1.06 / 1.04,
// six bits 4096 x 6656 / 4096 x 8192 1.10 / 1.15, five bits 4096 x 6144 / 4096 x 8192 / 8192 x 8192 0.98 / 1.05 / 1.13 (4096 x 8704 0.94); not where
// most lanes lack a second group and row ends are ragged (five and eight bits 12000 x 9000 0.87 / 0.96; eight bits 1024 x 20001 1.00), nor for one and two bits, which
// write little (4096 x 11008 0.95).  (Below the line 3000 x 7168, 13 MB at five bits and 16 at six, 1.05.)  Workgroups of eight and sixteen waves: a compute unit holds
// no more than four and two by their waves alone, and they are not held back further.
inline bool quantize_few_workgroups(int64_t rows, int64_t K, int bits, bool field)
{
    return bits > 2 && K % 128 == 0 && quantize_waves(rows, K, field) <= 4 && rows * round_up(K, kKPad) / 8 * (field ? 6 : bits) > 17000000;
}
hipError_t launch_unpack(const uint32_t *packed, int64_t rows, int64_t K, int bits, bool field, uint8_t *codes,
                         hipStream_t stream);

// Design B: plane pairs by XOR + popcount on the vector ALU (any p, q in 1..8).
hipError_t launch_gemm_valu(const GemmArgs &args, hipStream_t stream);

// Design A: planes recombined into E2M1 / E2M3 codes in registers, f8f6f4 MFMA, exact fp32 accumulate
// (p, q in 1..4 while 4 K (2^p - 1)(2^q - 1) < 2^24).
bool gemm_mfma_fp4_supported(const GemmArgs &args);
hipError_t launch_gemm_mfma_fp4(const GemmArgs &args, hipStream_t stream);

// Design A with K split across the four waves of a workgroup (apmm_gemm_mfma_ksplit.h): for outputs of few
// tiles; same widths and exactness bound as above.
bool gemm_mfma_ksplit_supported(const GemmArgs &args);
bool gemm_mfma_ksplit_pays(const GemmArgs &args);  // the launch rule of launch_gemm_mfma_fp4 takes it for these
hipError_t launch_gemm_mfma_ksplit(const GemmArgs &args, hipStream_t stream);

// Codes of more than four bits, and 3- and 4-bit codes at a K beyond the bound above: int8 operands (apmm_gemm_mfma_i8.h).
bool gemm_mfma_i8_supported(const GemmArgs &args);
hipError_t launch_gemm_mfma_i8(const GemmArgs &args, hipStream_t stream);

// Ablation kernels for the claim of paper Sec. 4.2 (apmm_gemm_ablation.hip): the planes as +-1 operands on the
// matrix unit.  pairs != nullptr: every plane pair's product to global memory (p q M N int32 at `pairs`), then a
// recovery pass; pairs == nullptr: one tile per workgroup, recovery in registers.
bool gemm_ablation_supported(const GemmArgs &args);
size_t gemm_ablation_pairs_bytes(const GemmArgs &args);
hipError_t launch_gemm_ablation(const GemmArgs &args, int32_t *pairs, hipStream_t stream);

// Measurement aid: a pair of events that the next GEMM launch of the calling thread (large-tile MFMA kernel or
// small-M kernels) attaches to its kernel dispatch (hipExtLaunchKernel), so that they hold the kernel's own
// begin and end.
struct KernelTiming {
    hipEvent_t start, stop;
};
void set_kernel_timing(hipEvent_t start, hipEvent_t stop);
KernelTiming take_kernel_timing();  // returns the pair and clears it
// Measurement aid: name (with template arguments) of the GEMM kernel the calling thread launched last.  The format and the arguments are kept
// and written out when the name is asked for: both are string literals, or int.  Every %d or %s takes the next argument, whatever its
// kind, and nothing where there is none left.
struct KernelNameArg {
    const char *text = nullptr;
    int number = 0;
};
inline KernelNameArg kernel_name_arg(int number) { return {nullptr, number}; }
inline KernelNameArg kernel_name_arg(const char *literal) { return {literal, 0}; }
constexpr int kMaxKernelNameArgs = 5;
void keep_kernel_name(const char *fmt, const KernelNameArg *args, int count);
template <class... Args>
inline void note_kernel(const char *fmt, Args... args)
{
    static_assert(sizeof...(Args) <= kMaxKernelNameArgs, "arguments of a kernel's name");
    static_assert(((std::is_same<Args, int>::value || std::is_same<Args, const char *>::value) && ...), "int or a literal");
    const KernelNameArg list[sizeof...(Args) + 1] = {kernel_name_arg(args)...};
    keep_kernel_name(fmt, list, (int)sizeof...(Args));
}
const char *last_kernel();

// Small-M weight-streaming kernels: on the fp4 matrix operations for p, q <= 4 (M <= 64; unpacked activation codes of 3 and 4
// bits: M <= 32), on the int8 ones where gemm_decode_i8_supported, XOR/popcount for what is left (M <= 16).
// gemm_decode_supported is what the public small-M algo covers; launch_gemm_decode takes both sets.
bool gemm_decode_supported(const GemmArgs &args);
hipError_t launch_gemm_decode(const GemmArgs &args, hipStream_t stream);
// The XOR/popcount small-M kernel whatever the code widths (M <= 16, q <= 4): design B at decode shapes.
bool gemm_decode_valu_supported(const GemmArgs &args);
hipError_t launch_gemm_decode_valu(const GemmArgs &args, hipStream_t stream);
// The int8 small-M kernels (apmm_gemm_decode_i8.h); `tt`: tiles of 16 tokens, 1, 2 or 4.
bool gemm_decode_i8_supported(const GemmArgs &args);
hipError_t launch_gemm_decode_i8(const GemmArgs *args, int count, int tt, hipStream_t stream);
// Up to kMaxGroup small-M problems of equal p, q in one launch; they must all be covered by the same
// kernel variant (gemm_decode_group_supported).
bool gemm_decode_group_supported(const GemmArgs *args, int count);
hipError_t launch_gemm_decode_group(const GemmArgs *args, int count, hipStream_t stream, bool xor_only = false);

}  // namespace apmm
