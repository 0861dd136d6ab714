"""The name of the last GEMM kernel is kept as a format and its arguments and written out when it is asked for (apmm_kernels.h): through
the library, on the host."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2409_17870_amd")

PROGRAM = r"""
#include <cstdio>
#include "apmm_kernels.h"
int main()
{
    apmm::note_kernel("plain");
    std::puts(apmm::last_kernel());
    apmm::note_kernel("k<%d,%s,%d>", 7, (const char *)"codes", -3);
    std::puts(apmm::last_kernel());
    std::puts(apmm::last_kernel());
    apmm::note_kernel("missing<%d,%d,%s>", 1);
    std::puts(apmm::last_kernel());
    apmm::note_kernel("kind<%s,%d>%", 2, (const char *)"t");
    std::puts(apmm::last_kernel());
    apmm::note_kernel("%s%s", (const char *)"0123456789012345678901234567890123456789012345678901234567890123456789",
                      (const char *)"0123456789012345678901234567890123456789");
    std::puts(apmm::last_kernel());
}
"""
WANT = ["plain", "k<7,codes,-3>", "k<7,codes,-3>", "missing<1,,>", "kind<2,t>", ("0123456789" * 10)[:95]]


def _compile(tmp_path, text):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if shutil.which(hipcc) is None:
        pytest.skip("no hipcc")
    if not os.path.exists(os.path.join(PKG, "libapmm.so")):
        import __graft_entry__
        __graft_entry__.build()
    (tmp_path / "name.hip").write_text(text)
    return subprocess.run([hipcc, "-O0", "-std=c++17", "--offload-host-only", "-I", os.path.join(PKG, "csrc"), str(tmp_path / "name.hip"), "-L", PKG,
                           "-l:libapmm.so", "-Wl,-rpath," + PKG, "-o", str(tmp_path / "name")], capture_output=True, text=True)


def test_names(tmp_path):
    done = _compile(tmp_path, PROGRAM)
    assert done.returncode == 0, done.stderr
    assert subprocess.run([str(tmp_path / "name")], capture_output=True, text=True, check=True).stdout.split("\n")[:-1] == WANT


@pytest.mark.parametrize("args", ["\"%ld\", 5L", "\"%s\", std::string(\"x\")", "\"%d%d%d%d%d%d\", 1, 2, 3, 4, 5, 6"])
def test_other_arguments_do_not_compile(tmp_path, args):
    done = _compile(tmp_path, "#include <string>\n#include \"apmm_kernels.h\"\nint main() { apmm::note_kernel(%s); }\n" % args)
    assert done.returncode != 0 and "static assertion failed" in done.stderr
