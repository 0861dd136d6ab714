"""What the compiler made of the kernels, read from the code objects inside the library (its own build): registers that did not
suffice show up as spills, which cost a kernel of a few microseconds more than a wrong tile."""
import os
import re
import struct

import pytest

msgpack = pytest.importorskip("msgpack")

BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"


def _notes(elf):
    """AMDGPU metadata notes of a code object."""
    table, = struct.unpack_from("<Q", elf, 40)
    entry, count = struct.unpack_from("<HH", elf, 58)
    for i in range(count):
        kind, = struct.unpack_from("<I", elf, table + i * entry + 4)
        at, size = struct.unpack_from("<QQ", elf, table + i * entry + 24)
        end = at + size if kind == 7 else at  # SHT_NOTE
        while at < end:
            name, desc, note = struct.unpack_from("<III", elf, at)
            at += 12 + (name + 3) // 4 * 4
            if note == 32:  # NT_AMDGPU_METADATA
                yield msgpack.unpackb(elf[at:at + desc])
            at += (desc + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    from paper_2409_17870_amd import binding
    if not os.path.exists(binding.LIB_PATH):
        import __graft_entry__
        __graft_entry__.build()
    data = open(binding.LIB_PATH, "rb").read()
    found = {}
    pos = data.find(BUNDLE)
    while pos >= 0:
        count, = struct.unpack_from("<Q", data, pos + 24)
        at = pos + 32
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", data, at)
            triple = data[at + 24:at + 24 + length]
            at += 24 + length
            if b"amdgcn" in triple and size:
                for meta in _notes(data[pos + offset:pos + offset + size]):
                    found.update((k[".name"], k) for k in meta["amdhsa.kernels"])
        pos = data.find(BUNDLE, pos + 24)
    assert found
    return found


def _of(kernels, name):
    """{template arguments: metadata} of a kernel template with integer and bool arguments."""
    out = {}
    for mangled, meta in kernels.items():
        m = re.search(r"%d%sI((?:L[ib]\d+E)+)E" % (len(name), name), mangled)
        if m:
            out[tuple(int(x) for x in re.findall(r"L[ib](\d+)E", m.group(1)))] = meta
    assert out, name
    return out


@pytest.mark.parametrize("name", ["gemm_mfma_ksplit_kernel", "gemm_decode_i8_kernel", "gemm_decode_mfma_kernel", "gemm_mfma_lds_kernel"])
def test_no_vector_register_is_spilled(kernels, name):
    spilled = {a: k[".vgpr_spill_count"] for a, k in _of(kernels, name).items() if k[".vgpr_spill_count"]}
    assert not spilled


@pytest.mark.parametrize("p", [1, 2])
@pytest.mark.parametrize("q", [1, 2, 3])
def test_few_tokens_from_codes_leave_three_workgroups_on_a_compute_unit(kernels, p, q):
    """gemm_decode_mfma_kernel<p, q, 1, 1, codes, one chunk per lane>: eight waves a workgroup and 512 registers to a lane of the
    four vector units (handed out in eights) make three workgroups up to 80 registers."""
    assert _of(kernels, "gemm_decode_mfma_kernel")[(p, q, 1, 1, 1, 1)][".vgpr_count"] <= 80


def test_only_tiles_that_a_launch_rule_names_are_built(kernels):
    """gemm_mfma_ksplit_kernel<P, Q, row blocks, column blocks>"""
    for p, q, wm, wn in _of(kernels, "gemm_mfma_ksplit_kernel"):
        if wm == 4:
            assert wn == 4 and q >= 2
        else:
            assert wm == 2 and wn in ((2, 4) if p <= 2 else (2, 4, 5, 6) if q <= 2 else (2, 4, 5))
