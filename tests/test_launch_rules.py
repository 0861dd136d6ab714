"""The launchers' rules, host functions of sizes, addresses and widths, compiled for the host alone and asked on both sides of their
lines: which calls store their inner tiles streaming, which quantise four rows to a workgroup, with how many waves to a row and which with few workgroups to a compute unit, which pack by eight rows, in which tiles through LDS one workgroup goes ahead, and which take the direct tiles or the register form of the 128 x 128 K split where the
kernels that share operands through LDS are slower."""
import os
import shutil
import subprocess

import pytest

from test_pack_eights import SHAPES as PACKED

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2409_17870_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "apmm_gemm_mfma_ksplit.h"
#include "apmm_gemm_mfma_tiles.h"
namespace apmm { KernelTiming take_kernel_timing() { return {}; } void note_kernel(const char *, ...) {} }
using namespace apmm;
using namespace apmm::mfma;
int main()
{
    long long M, N, K, i32, f16;
    char kind[32];
    while (std::scanf("%31s %lld %lld %lld %lld %lld", kind, &M, &N, &K, &i32, &f16) == 6) {
        GemmArgs g{};
        g.M = M; g.N = N; g.K = K;
        g.c_i32 = (int32_t *)i32; g.c_f16 = (uint16_t *)f16;
        const std::string k = kind;
        const int r = k == "direct" ? direct_streams(2, 2, g) : k == "direct42" ? direct_streams(4, 2, g) : k == "direct44" ? direct_streams(4, 4, g)
                    : k == "ksplit22" ? ksplit_streams(2, 2, g) : k == "ksplit25" ? ksplit_streams(2, 5, g) : k == "ksplit44" ? ksplit_streams(4, 4, g)
                    : k == "lds" ? lds_streams<2, 2, 2, 2, 1>(g) : k == "ldsW4A4" ? lds_streams<4, 4, 2, 2, 1>(g)
                    : k == "ldswide" ? lds_streams<4, 2, 2, 4, 1>(g) : k == "ldskg2" ? lds_streams<4, 4, 2, 2, 2>(g) : -1;
        const DirectTile t = k == "field41" ? field_direct_tile<4, 1>(g) : k == "field42" ? field_direct_tile<4, 2>(g) : k == "field33" ? field_direct_tile<3, 3>(g)
                           : k == "field44" ? field_direct_tile<4, 4>(g) : DirectTile{0, 0};
        auto rounds = [&](auto pays, int bm, int bn) { return (int)pays(g, bm, bn, tile_count(g, bm, bn)); };
        if (k.compare(0, 5, "field") == 0) std::printf("%d\n", 10 * t.wm + t.wn);
        else if (k == "r23") std::printf("%d\n", rounds(rounds_go_direct<2, 3>, 256, 256));
        else if (k == "r23half") std::printf("%d\n", rounds(rounds_go_direct<2, 3>, 256, 128));
        else if (k == "r24") std::printf("%d\n", rounds(rounds_go_direct<2, 4>, 256, 128));
        else if (k == "r14") std::printf("%d\n", rounds(rounds_go_direct<1, 4>, 128, 128));
        else if (k == "r22") std::printf("%d\n", rounds(rounds_go_direct<2, 2>, 256, 256));
        else if (k == "r11") std::printf("%d\n", rounds(rounds_go_direct<1, 1>, 256, 256));
        else if (k == "quant") std::printf("%d\n", (int)quantize_rows_by_four(M, K));
        else if (k == "few") std::printf("%d\n", (int)quantize_few_workgroups(M, K, (int)N, N == 3 || N == 4));
        else if (k == "waves" || k == "wavesf") std::printf("%d\n", quantize_waves(M, K, k == "wavesf"));
        else if (k.compare(0, 5, "ahead") == 0) {
            const int tiles = (int)M, kk = (int)K;
            const std::string v = k.substr(5);
            std::printf("%d\n", v == "11" ? (int)lds_goes_ahead<1, 1, 2>(tiles, kk) : v == "21" ? (int)lds_goes_ahead<2, 1, 2>(tiles, kk) : v == "12" ? (int)lds_goes_ahead<1, 2, 2>(tiles, kk)
                              : v == "24" ? (int)lds_goes_ahead<2, 4, 2>(tiles, kk) : v == "42" ? (int)lds_goes_ahead<4, 2, 2>(tiles, kk) : v == "42wide" ? (int)lds_goes_ahead<4, 2, 4>(tiles, kk)
                              : v == "33" ? (int)lds_goes_ahead<3, 3, 2>(tiles, kk) : v == "44" ? (int)lds_goes_ahead<4, 4, 2>(tiles, kk) : -1);
        }
        else if (k == "eights" || k == "eightsf") std::printf("%d\n", (int)pack_by_eights(M, K, (int)N, k == "eightsf"));
        else if (k == "max13") std::printf("%lld\n", (long long)ksplit_lds_max_k(1, 3, g));
        else if (k == "max23") std::printf("%lld\n", (long long)ksplit_lds_max_k(2, 3, g));
        else if (k == "max24") std::printf("%lld\n", (long long)ksplit_lds_max_k(2, 4, g));
        else if (k == "max44") std::printf("%lld\n", (long long)ksplit_lds_max_k(4, 4, g));
        else std::printf("%d\n", r);
    }
}
"""

AT = 1 << 20  # an address at a line; 0: no output
STREAMS = [
    # (kernel, M, N, K, int32 at, fp16 at, streams)
    ("direct", 512, 4098, 512, AT, 0, 1), ("direct", 512, 4098, 512, 0, AT, 1),         # one output: always
    ("direct", 1024, 4096, 512, AT, AT, 1), ("direct", 2048, 4096, 512, AT, AT, 0),     # whole lines, 25 and 50 MB
    ("direct", 203, 4098, 512, AT, AT, 0), ("direct", 512, 4098, 512, AT, AT, 1),       # parts of lines, 5 and 13 MB
    ("direct", 512, 8010, 512, AT, AT, 0), ("direct42", 512, 8010, 512, AT, AT, 1),     # 25 MB
    ("direct42", 1500, 4098, 512, AT, AT, 0), ("direct44", 512, 4096, 512, AT, AT, 0),
    ("direct", 203, 4096, 512, AT + 4, AT, 0), ("direct", 203, 4096, 512, AT, AT + 2, 0), ("direct", 203, 4096, 512, AT, AT + 64, 1),
    ("ksplit22", 128, 4098, 512, AT, AT, 0), ("ksplit22", 128, 4096, 512, AT, AT, 1), ("ksplit22", 128, 4098, 512, AT, 0, 1),
    ("ksplit25", 512, 5003, 512, AT, AT, 1), ("ksplit44", 2048, 1500, 11008, AT, AT, 0), ("ksplit44", 2048, 1504, 11008, AT, AT, 1),
    ("lds", 1500, 11010, 512, AT, AT, 0), ("lds", 1500, 11010, 512, AT, 0, 0), ("lds", 1500, 11010, 512, 0, AT, 0),
    ("lds", 1000, 2602, 512, AT, AT, 1),
    ("lds", 1000, 6512, 512, AT, 0, 1), ("lds", 1000, 6504, 512, AT, 0, 0),             # 26 MB of int32: half lines, parts of them
    ("lds", 2048, 11008, 1088, AT, AT, 1), ("lds", 2048, 11008, 1024, AT, AT, 0), ("lds", 2048, 11008, 512, AT, AT, 0), ("lds", 1024, 11008, 2048, AT, AT, 0),
    ("lds", 1024, 11008, 4096, AT, AT, 1), ("lds", 2048, 11008, 512, AT, 0, 0), ("lds", 2048, 11008, 513, AT, 0, 1), ("lds", 4096, 8192, 512, AT, 0, 1), ("lds", 2048, 11008, 512, 0, AT, 1),
    ("lds", 1024, 6144, 512, AT, AT, 1),
    ("ldsW4A4", 2048, 11008, 512, AT, AT, 1), ("ldsW4A4", 1024, 11008, 512, AT, AT, 0),
    ("ldsW4A4", 1024, 11016, 5999, AT, AT, 0), ("ldsW4A4", 1024, 11016, 6000, AT, AT, 1), ("ldswide", 2048, 11016, 6000, AT, AT, 0),
    ("ldskg2", 1024, 3000, 4096, AT, 0, 1), ("ldskg2", 1024, 3000, 4096, AT, AT, 1), ("ldskg2", 512, 2050, 4096, AT, AT, 0),
]
# (rule, M, N, K, int32 at, fp16 at, answer): the direct tile's wave rows and columns, or whether several rounds go to the direct tile
RULES = [
    ("field41", 1024, 2048, 4096, AT, 0, 14), ("field41", 1024, 2048, 4096, 0, AT, 0), ("field41", 1024, 2048, 2560, 0, AT, 14),
    ("field41", 2048, 2048, 2560, 0, AT, 0), ("field41", 2048, 2048, 1024, AT, AT, 14), ("field41", 2048, 2048, 2048, AT, AT, 0),
    ("field41", 512, 3000, 2048, AT, AT, 14), ("field41", 2048, 2176, 1024, AT, 0, 0), ("field41", 2048, 2048, 10240, 0, AT, 14),
    ("field42", 1024, 2048, 2048, AT, 0, 14), ("field42", 1024, 2176, 2048, AT, 0, 0), ("field42", 1024, 2048, 3072, AT, 0, 0),
    ("field42", 1024, 2048, 2048, 0, AT, 0), ("field42", 1024, 2048, 2047, 0, AT, 14),
    ("field33", 512, 4096, 1024, AT, 0, 22), ("field33", 768, 4096, 1024, AT, 0, 0), ("field33", 768, 4096, 512, AT, 0, 22),
    ("field33", 512, 4096, 512, 0, AT, 0), ("field33", 2048, 4096, 8192, 0, AT, 24), ("field33", 2048, 4096, 8191, 0, AT, 0),
    ("field33", 2048, 4096, 8192, AT, AT, 0), ("field33", 2048, 3328, 8192, 0, AT, 0), ("field33", 2048, 4352, 8192, 0, AT, 0),
    ("field44", 512, 4096, 512, AT, 0, 0), ("field44", 2048, 4096, 11008, 0, AT, 0),
    ("r23", 4096, 8192, 4096, 0, AT, 1), ("r23", 4096, 8192, 4095, 0, AT, 0), ("r23", 4096, 8192, 8191, AT, AT, 0),
    ("r23", 4096, 8192, 8192, AT, AT, 1), ("r23", 4096, 11008, 8191, AT, 0, 0), ("r23", 4096, 11008, 8192, AT, 0, 1),
    ("r23", 4096, 5120, 11008, AT, 0, 0), ("r23half", 2048, 11008, 8192, 0, AT, 1), ("r23half", 2048, 11008, 8192, AT, AT, 0),
    ("r24", 4096, 4096, 6144, 0, AT, 1), ("r24", 4096, 4096, 6143, 0, AT, 0), ("r24", 4096, 4096, 10240, AT, AT, 1),
    ("r24", 4096, 8192, 11008, 0, AT, 0), ("r14", 600, 13824, 11008, AT, 0, 1), ("r14", 700, 11008, 11008, AT, 0, 0),
    ("r14", 700, 11008, 8192, AT, 0, 1), ("r14", 1024, 11008, 8192, AT, 0, 0), ("r14", 600, 13824, 4095, AT, 0, 0),
    ("r22", 4096, 8192, 8192, 0, AT, 1), ("r22", 4096, 8192, 8192, AT, 0, 0), ("r22", 4096, 8192, 10240, AT, 0, 1), ("r11", 4096, 8192, 8192, 0, AT, 0),
    ("r11", 4096, 8192, 512, 0, AT, 1), ("r11", 4096, 8192, 512, AT, 0, 0), ("r11", 4096, 8192, 513, 0, AT, 0), ("r11", 8192, 8192, 512, 0, AT, 0),
    ("quant", 512, 0, 8192, 0, 0, 0), ("quant", 513, 0, 8192, 0, 0, 1), ("quant", 1024, 0, 2048, 0, 0, 0), ("quant", 1225, 0, 2048, 0, 0, 1),
    ("quant", 640, 0, 4096, 0, 0, 1), ("quant", 610, 0, 4096, 0, 0, 0), ("quant", 641, 0, 4300, 0, 0, 0), ("quant", 900, 0, 4300, 0, 0, 1),
    ("quant", 513, 0, 4900, 0, 0, 0), ("quant", 800, 0, 4900, 0, 0, 1), ("quant", 513, 0, 8704, 0, 0, 0), ("quant", 641, 0, 8704, 0, 0, 1),
    ("quant", 1024, 0, 2560, 0, 0, 1), ("quant", 1025, 0, 2560, 0, 0, 0), ("quant", 1599, 0, 2049, 0, 0, 0), ("quant", 1600, 0, 2049, 0, 0, 1),
    ("quant", 1300, 0, 2561, 0, 0, 1), ("quant", 513, 0, 16384, 0, 0, 1), ("quant", 4096, 0, 16385, 0, 0, 0),
    ("few", 4096, 8, 4096, 0, 0, 0), ("few", 4151, 8, 4096, 0, 0, 1), ("few", 4150, 8, 4096, 0, 0, 0), ("few", 4096, 5, 6912, 0, 0, 1), ("few", 4096, 5, 6144, 0, 0, 0),
    ("few", 12000, 8, 9000, 0, 0, 0), ("few", 2048, 8, 20000, 0, 0, 0), ("few", 2048, 4, 20000, 0, 0, 0), ("few", 2048, 8, 11008, 0, 0, 0), ("few", 2048, 8, 10240, 0, 0, 1), ("few", 1024, 8, 20001, 0, 0, 0),  # eight waves to a row; ragged
    ("few", 16384, 2, 11008, 0, 0, 0),
    ("waves", 1, 0, 2048, 0, 0, 1), ("waves", 4096, 0, 2049, 0, 0, 2), ("waves", 4096, 0, 4097, 0, 0, 4), ("waves", 1, 0, 8192, 0, 0, 4), ("waves", 1, 0, 8193, 0, 0, 8),
    ("wavesf", 1024, 0, 8704, 0, 0, 8), ("wavesf", 1025, 0, 8704, 0, 0, 4), ("wavesf", 1025, 0, 10240, 0, 0, 4), ("wavesf", 1025, 0, 10752, 0, 0, 8),
    ("waves", 256, 0, 11008, 0, 0, 8), ("waves", 257, 0, 11008, 0, 0, 4), ("waves", 2047, 0, 16384, 0, 0, 4), ("waves", 2048, 0, 16384, 0, 0, 8), ("waves", 2048, 0, 10240, 0, 0, 4),
    ("waves", 1, 0, 16384, 0, 0, 8), ("waves", 256, 0, 16385, 0, 0, 16), ("waves", 257, 0, 16896, 0, 0, 8),
    ("waves", 768, 0, 9000, 0, 0, 8), ("waves", 769, 0, 9000, 0, 0, 4), ("waves", 4096, 0, 16383, 0, 0, 4), ("waves", 1024, 0, 16383, 0, 0, 4),  # rows that end in a k block
    ("waves", 1024, 0, 20001, 0, 0, 4), ("waves", 1024, 0, 22527, 0, 0, 4), ("waves", 1024, 0, 22529, 0, 0, 8), ("waves", 1025, 0, 16385, 0, 0, 8), ("waves", 769, 0, 16896, 0, 0, 8),
    ("waves", 8388544, 0, 11008, 0, 0, 8), ("waves", 8388545, 0, 11008, 0, 0, 4), ("waves", 16000000, 0, 20480, 0, 0, 4),  # 2^32 work items of a launch
    ("eights", 536870880, 3, 64, 0, 0, 1), ("eights", 536870912, 3, 64, 0, 0, 0), ("eights", 67108832, 8, 4000, 0, 0, 1), ("eights", 67108864, 8, 4000, 0, 0, 0),  # 2^32 work items
    ("eights", 600000000, 2, 200, 0, 0, 0), ("eightsf", 536870880, 4, 3, 0, 0, 1), ("eightsf", 536870912, 4, 3, 0, 0, 0), ("eights", 178956960, 5, 1400, 0, 0, 1), ("eights", 178956992, 5, 1400, 0, 0, 0),
    ("eights", 5003, 3, 3001, 0, 0, 1), ("eightsf", 2048, 4, 4096, 0, 0, 1), ("eights", 1000, 3, 4096, 0, 0, 0), ("eights", 1700, 3, 3300, 0, 0, 1), ("eights", 1699, 3, 3300, 0, 0, 0),
    ("eights", 1700, 3, 3299, 0, 0, 0), ("eights", 2049, 3, 4096, 0, 0, 0), ("eights", 3071, 3, 4096, 0, 0, 0), ("eights", 3300, 3, 4096, 0, 0, 1), ("eights", 4200, 3, 4096, 0, 0, 0),
    ("eights", 5003, 3, 1998, 0, 0, 0), ("eights", 6144, 3, 733, 0, 0, 1), ("eights", 6144, 3, 732, 0, 0, 0), ("eights", 9001, 3, 511, 0, 0, 1),
    ("eights", 2048, 5, 5120, 0, 0, 1), ("eights", 1920, 5, 5120, 0, 0, 0), ("eights", 1921, 5, 5120, 0, 0, 1), ("eights", 3872, 5, 5120, 0, 0, 0), ("eights", 3873, 5, 5120, 0, 0, 1), ("eights", 5376, 5, 5120, 0, 0, 0), ("eights", 2500, 5, 11008, 0, 0, 0), ("eights", 5003, 5, 11008, 0, 0, 0), ("eights", 5504, 5, 11008, 0, 0, 1),
    ("eights", 11008, 6, 8192, 0, 0, 0), ("eights", 11008, 6, 7000, 0, 0, 1), ("eightsf", 11008, 4, 8192, 0, 0, 0), ("eights", 11008, 4, 8192, 0, 0, 1),
    ("eights", 2048, 2, 24576, 0, 0, 1), ("eights", 2500, 2, 24576, 0, 0, 0), ("eights", 8192, 2, 5120, 0, 0, 0), ("eights", 8192, 1, 12207, 0, 0, 0), ("eights", 8192, 1, 12208, 0, 0, 1),
    ("ahead42wide", 688, 0, 2048, 0, 0, 1), ("ahead42wide", 688, 0, 2047, 0, 0, 0), ("ahead42wide", 512, 0, 4096, 0, 0, 0), ("ahead42wide", 737, 0, 4096, 0, 0, 0),
    ("ahead42", 513, 0, 4096, 0, 0, 1), ("ahead42", 513, 0, 4095, 0, 0, 0), ("ahead33", 736, 0, 2048, 0, 0, 1), ("ahead33", 736, 0, 2047, 0, 0, 0), ("ahead44", 736, 0, 2560, 0, 0, 1),
    ("ahead44", 736, 0, 2559, 0, 0, 0), ("ahead11", 1032, 0, 4096, 0, 0, 0), ("ahead21", 1032, 0, 2048, 0, 0, 1), ("ahead12", 961, 0, 4096, 0, 0, 1), ("ahead12", 960, 0, 4096, 0, 0, 0),
    ("ahead12", 1105, 0, 4096, 0, 0, 0), ("ahead24", 1032, 0, 4096, 0, 0, 0),
    ("max13", 1, 1, 1, AT, 0, 8192), ("max13", 1, 1, 1, 0, AT, 9216), ("max23", 1, 1, 1, AT, 0, 5632), ("max23", 1, 1, 1, AT, AT, 8704),
    ("max24", 1, 1, 1, AT, 0, 7168), ("max44", 1, 1, 1, AT, 0, 9216),
]
CASES = STREAMS + RULES + [("eightsf" if kind == "a" and bits in (3, 4) else "eights", rows, bits, K, 0, 0, by_eights) for kind, bits, rows, K, by_eights in PACKED]


@pytest.fixture(scope="module")
def answers(tmp_path_factory):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if shutil.which(hipcc) is None:
        pytest.skip("no hipcc")
    d = tmp_path_factory.mktemp("rule")
    (d / "rule.hip").write_text("#include <string>\n" + PROGRAM)
    subprocess.run([hipcc, "-O0", "-std=c++17", "--offload-host-only", "-I", CSRC, str(d / "rule.hip"), "-o", str(d / "rule")], check=True,
                   capture_output=True)
    lines = "".join("%s %d %d %d %d %d\n" % c[:6] for c in CASES)
    return [int(x) for x in subprocess.run([str(d / "rule")], input=lines, capture_output=True, text=True, check=True).stdout.split()]


@pytest.mark.parametrize("i", range(len(CASES)))
def test_rule(answers, i):
    assert answers[i] == CASES[i][6], CASES[i]
