"""Registers of the update's kernels, from the metadata of the built library: where sums leave cell by cell, three sums of 8
workers and two of 4 keep four wavefronts on a SIMD (128 registers each), which the code that sends pairs of cells would cost
them."""
import os
import re

import pytest

from paper_1903_04488_amd import binding


def _registers():
    """vector registers by (mangled) kernel name"""
    if not os.path.exists(binding.library_path()):
        pytest.skip("the library is not built")
    with open(binding.library_path(), "rb") as f:
        code = f.read()
    found = {}
    for m in re.finditer(rb"\xab\.vgpr_count(?:([\x00-\x7f])|\xcc(.)|\xcd(..))", code, re.S):
        at = code.rfind(b"\xa5.name", 0, m.start()) + 6
        size, start = {0xd9: (code[at + 1], at + 2), 0xda: (code[at + 1] << 8 | code[at + 2], at + 3)}.get(code[at], (code[at] & 31, at + 1))
        found[code[start:start + size].decode()] = int.from_bytes(m.group(1) or m.group(2) or m.group(3), "big")
    return found


@pytest.mark.parametrize("lanes,wavefronts,sums", [(8, 4, 2), (8, 4, 3), (4, 1, 2)])
def test_cell_by_cell_keeps_four_wavefronts_on_a_simd(lanes, wavefronts, sums):
    start = f"k_accumulate_visitsILi{lanes}ELi16ELi{wavefronts}ELi{sums}ELb0E"
    those = {name: n for name, n in _registers().items() if re.search(start + r"(Lb0E)?NS0_9VisitRowsE", name)}
    assert len(those) == 1
    assert max(those.values()) <= 128
