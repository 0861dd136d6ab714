"""Tile maps divide by a multiplication with the reciprocal that the launcher passes (apmm_mfma_common.h): the reciprocals, formed by the
launcher's own function on the host, against integer division."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2409_17870_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "apmm_mfma_common.h"
int main()
{
    long long d, most;
    while (std::scanf("%lld %lld", &d, &most) == 2) std::printf("%u\n", apmm::mfma::divisor_magic(d, most));
}
"""

# (divisor, all dividends lie below this)
PAIRS = [(d, most) for d in (1, 2, 3, 5, 7, 31, 32, 43, 172, 255, 641, 4096, 65535, 65536, 65537, 1 << 20)
         for most in (1, 2, 255, 4096, 65535, 65536, 65537, 1 << 20, (1 << 31) - 1)]


def test_reciprocals_of_divisors(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if shutil.which(hipcc) is None:
        pytest.skip("no hipcc")
    (tmp_path / "magic.hip").write_text(PROGRAM)
    subprocess.run([hipcc, "-O0", "-std=c++17", "--offload-host-only", "-I", CSRC, str(tmp_path / "magic.hip"), "-o", str(tmp_path / "magic")],
                   check=True, capture_output=True)
    lines = "".join("%d %d\n" % p for p in PAIRS)
    got = subprocess.run([str(tmp_path / "magic")], input=lines, capture_output=True, text=True, check=True).stdout.split()
    for (d, most), magic in zip(PAIRS, map(int, got)):
        if d == 1 or d * most >= 1 << 32:
            assert magic == 0, (d, most)         # the kernel divides
            continue
        edges = {x for k in range(0, most, max(1, most // 500)) for x in (k, k // d * d, k // d * d - 1, k // d * d + d - 1)} | {most - 1}
        for x in edges:
            if 0 <= x < most:
                assert (x * magic) >> 32 == x // d, (d, most, x)
