"""Packing of many rows (eight to a workgroup) against that of the same rows 32 at a time (a wave per tile or per row): the same bytes and code
sums, for every stored form, ragged rows and row ends, and on both sides of the rule's lines."""
import pytest
import torch

from paper_2409_17870_amd import binding

pytestmark = pytest.mark.gpu


# (weights or activations, bits, rows, K, whether the rule takes eight rows to a workgroup: held by the test of the launch rules)
SHAPES = [
    ("w", 3, 1500, 3001, 0), ("w", 4, 1531, 3008, 0), ("w", 5, 2048, 2499, 0), ("w", 6, 1633, 4096, 0), ("w", 7, 4500, 1001, 0),
    ("w", 8, 1503, 3200, 0), ("a", 3, 9001, 511, 1), ("a", 4, 2048, 4096, 1), ("a", 4, 1601, 3333, 0), ("a", 8, 1700, 5003, 0),
    ("a", 4, 1499, 4096, 0), ("w", 2, 10003, 4001, 0), ("w", 2, 2049, 20000, 0), ("w", 1, 33000, 3072, 1), ("w", 3, 1500003, 3, 1),
    ("a", 4, 1500001, 3, 1), ("w", 3, 1793, 3301, 1), ("w", 3, 5003, 3001, 1), ("w", 4, 2017, 4736, 1), ("w", 4, 3271, 3085, 1),
    ("w", 5, 6145, 801, 1), ("w", 6, 2041, 4097, 1), ("w", 7, 1705, 3400, 1), ("w", 8, 1953, 4223, 1), ("a", 3, 1930, 4100, 1),
    ("a", 4, 2016, 4999, 1), ("a", 8, 3300, 3100, 1), ("w", 2, 2048, 22001, 1), ("w", 1, 8191, 12300, 1),
    ("w", 3, 2016, 4672, 1), ("w", 7, 1984, 4160, 1), ("w", 8, 2048, 3328, 1), ("w", 2, 3840, 12032, 1),
]


def tiles_and_sums(packed, rows, K, slots):
    blocks, nkb = (rows + 31) // 32, (K + 511) // 512 * 4
    words = packed.view(torch.int32)
    n = blocks * nkb * slots * 128
    return words[:n].view(blocks, -1), words[n:n + 32 * blocks].view(blocks, 32)


@pytest.mark.parametrize("kind, bits, rows, K, by_eights", SHAPES)
def test_many_rows(kind, bits, rows, K, by_eights):
    g = torch.Generator(device="cuda").manual_seed(rows)
    whole = torch.randint(0, 256, (rows * K + 16,), generator=g, device="cuda", dtype=torch.uint8)  # high bits beyond the code are masked away
    slots = 6 if kind == "a" and bits in (3, 4) else bits
    pack = binding.apmm_pack_activations if kind == "a" else binding.apmm_pack_weights
    size = binding.apmm_packed_activation_bytes if kind == "a" else binding.apmm_packed_bytes
    for offset in (0, 3):
        codes = whole[offset:offset + rows * K].view(rows, K)
        tiles, sums = tiles_and_sums(pack(codes, bits, out=torch.full((size(rows, K, bits),), 165, device="cuda", dtype=torch.uint8)), rows, K, slots)
        last = (rows - 1) // 32
        for rb in sorted({0, 1, last // 3, last // 2 + 1, last - 1, last}):
            part = codes[32 * rb:32 * rb + 32].clone()
            t, s = tiles_and_sums(pack(part, bits, out=torch.zeros(size(len(part), K, bits), device="cuda", dtype=torch.uint8)), len(part), K, slots)
            assert torch.equal(tiles[rb], t[0]) and torch.equal(sums[rb], s[0]), (rb, offset)
