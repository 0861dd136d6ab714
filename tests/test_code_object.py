"""What the compiler made of the kernels, read from the code objects inside the library (its own build): registers that did not
suffice show up as spills, which cost a kernel of a few microseconds more than a wrong tile."""
import collections
import os
import re
import shutil
import struct
import subprocess

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
def code_objects():
    from paper_2409_17870_amd import binding
    if not os.path.exists(binding.LIB_PATH):
        import __graft_entry__
        __graft_entry__.build()
    data = open(binding.LIB_PATH, "rb").read()
    found = []
    pos = data.find(BUNDLE)
    while pos >= 0:
        count, = struct.unpack_from("<Q", data, pos + 24)
        at = pos + 32
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", data, at)
            triple = data[at + 24:at + 24 + length]
            at += 24 + length
            if b"amdgcn" in triple and size:
                found.append(data[pos + offset:pos + offset + size])
        pos = data.find(BUNDLE, pos + 24)
    return found


@pytest.fixture(scope="module")
def kernels(code_objects):
    found = {k[".name"]: k for elf in code_objects for meta in _notes(elf) for k in meta["amdhsa.kernels"]}
    assert found
    return found


@pytest.fixture(scope="module")
def dword_stores(code_objects, tmp_path_factory):
    """{mangled kernel name: Counter(plain=, nt=, pair=, behind=)} of the dword stores of the tiled kernels: streaming ones of two fp16 results (nt and
    pair), and of those the ones that follow another within three instructions (behind)"""
    objdump = shutil.which("llvm-objdump", path="/opt/rocm/llvm/bin" + os.pathsep + os.environ.get("PATH", ""))
    if objdump is None:
        pytest.skip("no llvm-objdump")
    path = str(tmp_path_factory.mktemp("co") / "kernels.co")
    found = {}
    for elf in code_objects:
        if b"gemm_mfma_" not in elf:
            continue
        with open(path, "wb") as f:
            f.write(elf)
        text = subprocess.run([objdump, "-d", "--no-show-raw-insn", path], capture_output=True, text=True, check=True).stdout
        count = None
        for line in text.splitlines():
            m = re.match(r"[0-9a-f]+ <(.*)>:$", line)
            if m:
                count = found[m.group(1)] = collections.Counter()
                pairs, since = set(), 99  # registers that a byte permute wrote last, instructions since the last store of one
            elif count is not None and line.startswith("\t"):
                since += 1
                op, args = (line.split("//")[0].split(None, 1) + [""])[:2]
                if op == "global_store_dword":
                    nt = args.rstrip().endswith(" nt")
                    count["nt" if nt else "plain"] += 1
                    if nt and args.split(", ")[1] in pairs:
                        count["pair"] += 1
                        count["behind"] += since <= 3
                        since = 0
                elif op.startswith("v_"):
                    to = args.split(",")[0].strip()
                    (pairs.add if op.startswith("v_perm_b32") else pairs.discard)(to)
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


@pytest.mark.parametrize("name", ["gemm_mfma_ksplit_kernel", "gemm_mfma_ksplit_long_kernel", "gemm_mfma_ksplit_wide_kernel", "gemm_decode_i8_kernel", "gemm_decode_mfma_kernel",
                                  "gemm_mfma_lds_kernel", "gemm_mfma_i8_kernel", "gemm_mfma_direct_kernel"])
def test_no_vector_register_is_spilled(kernels, name):
    """But for the 256 x 256 tile of single bits on both sides in one phase, which keeps 16 in scratch."""
    spilled = {a: k[".vgpr_spill_count"] for a, k in _of(kernels, name).items() if k[".vgpr_spill_count"]}
    if name == "gemm_mfma_direct_kernel":
        assert spilled.pop((1, 1, 4, 4, 1), 0) <= 16
    assert not spilled


def test_packing_and_quantising_kernels_spill_nothing(kernels):
    """pack_kernel is bound to eight waves to a vector unit, 64 registers."""
    found = {name: k for name, k in kernels.items() if re.search(r"\d(un)?pack_(rows_)?kernel|quantize_(pack|fields)_kernel", name)}
    assert len(found) == 10 + 4 + 12 + 8 + 1
    assert not [name for name, k in found.items() if k[".vgpr_spill_count"] or k[".private_segment_fixed_size"]]
    assert all(k[".vgpr_count"] <= 64 for name, k in found.items() if "11pack_kernel" in name)


@pytest.mark.parametrize("p", [1, 2])
@pytest.mark.parametrize("q", [1, 2, 3])
def test_few_tokens_from_codes_leave_three_workgroups_on_a_compute_unit(kernels, p, q):
    """gemm_decode_mfma_kernel<p, q, 1, 1, codes, one chunk per lane>: eight waves a workgroup and 512 registers to a lane of the
    four vector units (handed out in eights) make three workgroups up to 80 registers."""
    assert _of(kernels, "gemm_decode_mfma_kernel")[(p, q, 1, 1, 1, 1)][".vgpr_count"] <= 80


@pytest.mark.parametrize("p", [1, 2, 3, 4])
@pytest.mark.parametrize("q", [1, 2, 3, 4])
def test_17_to_32_tokens_from_codes_leave_two_workgroups_on_a_compute_unit(kernels, p, q):
    """gemm_decode_mfma_kernel<p, q, 2, channel tiles, aligned codes, 8>: two workgroups up to 128 registers.  Not 4-bit weights under field-form
    codes, and not single-bit codes under 2-bit weights with two channel tiles, where one register is missing."""
    of = _of(kernels, "gemm_decode_mfma_kernel")
    if p <= 2 or q < 4:
        assert of[(p, q, 2, 1, 1, 8)][".vgpr_count"] <= 128
    if p <= 2 and q <= 2 and (p, q) != (1, 2):
        assert of[(p, q, 2, 2, 1, 8)][".vgpr_count"] <= 128


@pytest.mark.parametrize("q,registers", [(1, 144), (2, 140), (3, 148), (4, 144), (8, 148)])
def test_lane_addresses_of_four_token_tiles(kernels, q, registers):
    """gemm_decode_i8_kernel<nibbles, q, 4, 1>: three 64-bit lane addresses in the k loop, not six (six more registers and up to a tenth of the time)."""
    assert _of(kernels, "gemm_decode_i8_kernel")[(5, q, 4, 1)][".vgpr_count"] <= registers


def test_only_tiles_that_a_launch_rule_names_are_built(kernels):
    """gemm_mfma_ksplit_kernel<P, Q, row blocks, column blocks>, gemm_mfma_ksplit_long_kernel<P, Q>, gemm_mfma_ksplit_wide_kernel<P, Q>, gemm_mfma_lds_kernel<P, Q, row blocks,
    column blocks of a wave, waves to a vector unit> and gemm_mfma_direct_kernel<P, Q, row blocks, column blocks of a wave, phases>"""
    for p, q, wm, wn in _of(kernels, "gemm_mfma_ksplit_kernel"):
        if wm == 4:
            assert wn == 4 and q >= 2
        else:
            assert wm == 2 and wn in ((2, 4) if p <= 2 else (2, 4, 5, 6) if q <= 2 else (2, 4, 5))
    assert set(_of(kernels, "gemm_mfma_ksplit_long_kernel")) == {(p, q) for p in (1, 2, 3, 4) for q in (3, 4)}
    assert set(_of(kernels, "gemm_mfma_ksplit_wide_kernel")) == {(3, 2), (4, 2)}
    for p, q, wm, wn, _ in _of(kernels, "gemm_mfma_lds_kernel"):
        assert (wm, wn) == (2, 2) or (p > 2 and q <= 2 and (wm, wn) == (2, 4))
    for p, q, wm, wn, phases in _of(kernels, "gemm_mfma_direct_kernel"):
        if p > 2:
            assert phases == 1 and (wm, wn) in (((1, 4),) if q <= 2 else ((2, 2), (2, 4)) if q == 3 else ())
        else:
            assert (wm, wn) in ((4, 4), (4, 2), (2, 4), (2, 2)) and (q < 4 or (wm, wn) != (4, 4))
            assert phases == 1 or ((wm, wn) == (4, 4) and phases <= (3 if q == 1 else 2 if q == 2 else 1))


@pytest.mark.parametrize("name", ["gemm_mfma_i8_kernel", "gemm_mfma_lds_kernel", "gemm_mfma_direct_kernel", "gemm_mfma_ksplit_kernel",
                                  "gemm_mfma_ksplit_long_kernel"])
def test_inner_tiles_have_streaming_and_plain_stores(dword_stores, name):
    """A block of 32 x 32 takes 16 dword stores a lane of int32 and 8 of fp16 in pairs.  Every inner tile has both in a streaming and in a
    plain form (rows that are no whole lines), the border has int32 in plain stores: 24 streaming to 40 plain.  Two forms that
    differ in the hint alone are one to the compiler unless it is kept from joining them."""
    for args, count in _of(dword_stores, name).items():
        if name == "gemm_mfma_direct_kernel" and args[4] > 1:
            continue                                     # two phases: int32 in whole tiles alone
        if name == "gemm_mfma_ksplit_kernel" and args[2:] in ((2, 5), (2, 6)):
            assert count["nt"] * 2 == count["plain"] * 3  # outputs of a size that always streams: the border alone is plain
            continue
        assert count["nt"] > 0 and count["nt"] * 5 == count["plain"] * 3, (args, count)


def test_128_by_256_tile_stores_fp16_alone(dword_stores):
    """Four blocks a wave, 8 dword stores of pairs each, streaming and plain; no int32 store, which the launch rule never asks for."""
    for args, count in _of(dword_stores, "gemm_mfma_ksplit_wide_kernel").items():
        assert count["nt"] == count["plain"] == 32, (args, count)


@pytest.mark.parametrize("name", ["gemm_mfma_lds_kernel", "gemm_mfma_direct_kernel"])
def test_streaming_fp16_pairs_leave_together(kernels, dword_stores, name):
    """The pieces of 64 bytes that make up a row's line: further apart, fewer of them are joined on their way to memory."""
    seen = 0
    for (p, q, wm, wn, last), meta in _of(kernels, name).items():
        count = dword_stores[meta[".name"]]
        if wm * wn == 16 or (name == "gemm_mfma_direct_kernel" and last > 1):
            continue  # (with other operations, for want of registers; int32 output alone)
        seen += 1
        assert count["pair"] >= 8 * wm * wn and count["behind"] * wn >= 0.9 * count["pair"] * (wn - 1), (p, q, wm, wn, count)
    assert seen
