"""include/csketch.h is accepted by strict compilers of every C standard that it needs nothing newer than, and of C++, and cs_params
is as large for each of them as its mirror in the binding."""
import ctypes
import os
import subprocess

import pytest

from paper_1903_04488_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("std", ["c90", "c99", "c11", "c17", "c++98", "c++17"])
def test_header_compiles_strictly_and_keeps_its_layout(std, tmp_path):
    cpp = std.startswith("c++")
    src = tmp_path / ("header.cc" if cpp else "header.c")
    src.write_text("#include <stddef.h>\n#include \"csketch.h\"\n"
                   f"typedef char size[sizeof(cs_params) == {ctypes.sizeof(binding.CsParams)} ? 1 : -1];\n"
                   f"typedef char place[offsetof(cs_params, anyc) == {binding.CsParams.anyc.offset} ? 1 : -1];\n")
    # (c90 and C++98 get 64-bit numbers from the headers of the library, as extensions)
    subprocess.check_call(["g++" if cpp else "gcc", f"-std={std}", *(["-pedantic-errors"] if std not in ("c90", "c++98") else []),
                           "-Werror", "-fsyntax-only", "-I", os.path.join(ROOT, "include"), str(src)])
