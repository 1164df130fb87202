"""The bitmaps of a detection tile that the kernels also read as 64-bit rows lie on 8-byte
boundaries of the LDS, in every instantiation (offsets printed by a host build of the header)."""
import os
import re
import subprocess

import pytest

from paper_1008_2192_amd import build

PROGRAM = r"""
#include <stddef.h>
#include <stdio.h>
#include "detect_tile.h"
template <class L> void show() {
    printf("code %zu con_map %zu align %zu\n", offsetof(L, code), offsetof(L, con_map), alignof(L));
}
int main() {
    using namespace crb;
    show<DetectLds<16, 4, false>>();
    show<DetectLds<32, 4, false>>();
    show<DetectLds<64, 4, false>>();
    show<DetectLds<32, 6, true>>();
}
"""


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="needs hipcc")
def test_rows_of_64_bits_are_aligned(tmp_path):
    src, exe = tmp_path / "layout.hip", tmp_path / "layout"
    src.write_text(PROGRAM)
    subprocess.run([build.HIPCC, "--offload-arch=" + build.ARCH, "--offload-host-only", "-std=c++17",
                    "-Wno-invalid-offsetof", "-I", build.CSRC, str(src), "-o", str(exe)],
                   check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    lines = subprocess.run([str(exe)], check=True, stdout=subprocess.PIPE,
                           text=True).stdout.splitlines()
    assert len(lines) == 4
    for line in lines:
        code, con_map, align = map(int, re.findall(r"\d+", line))
        assert align % 8 == 0 and code % 8 == 0 and con_map % 8 == 0, line
