"""The kernels' check of a chunk-table entry (zipmoe_extent.h), built as host code, against the same in arithmetic that can not wrap."""
import itertools
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include <cinttypes>
#include <cstdio>
#include "zipmoe_extent.h"
int main()
{
    uint64_t chunk, a, b, e_offset, e_size;
    int raw;
    while (std::scanf("%d %" SCNu64 " %" SCNu64 " %" SCNu64 " %" SCNu64 " %" SCNu64, &raw, &chunk, &a, &b, &e_offset, &e_size) == 6)
        std::puts((raw ? zipmoe::raw_stream_inside(chunk, a, static_cast<uint32_t>(b), e_offset, e_size)
                       : zipmoe::stream_inside(chunk, static_cast<uint32_t>(a), static_cast<uint32_t>(b), e_offset, e_size)) ? "1" : "0");
}
"""


@pytest.fixture(scope="module")
def inside(tmp_path_factory):
    at = tmp_path_factory.mktemp("extent")
    (at / "extent.cpp").write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2601_21198_amd", "csrc"), "-I", os.path.join(ROOT, "include"),
                           str(at / "extent.cpp"), "-o", str(at / "extent")])

    def ask(cases):
        text = "\n".join(" ".join(str(x) for x in c) for c in cases)
        return [x == "1" for x in subprocess.run([str(at / "extent")], input=text, capture_output=True, text=True, check=True).stdout.split()]
    return ask


CHUNKS = [0, 16, 4080, 4096, 4112, 8192, 12272, 12288, 12304, (1 << 32) - 16, (1 << 63), (1 << 64) - 8192, (1 << 64) - 16]
REGIONS = [(4096, 0), (4096, 64), (4096, 8192), (4096, (1 << 32) + 64), (1 << 40, 8192), ((1 << 64) - 8192, 8191)]


def test_coded_streams(inside):
    offsets = [0, 16, 63, 64, 65, 80, 4096, 8127, 8128, 8192, 8193, (1 << 31), (1 << 32) - 64, (1 << 32) - 16, (1 << 32) - 1]
    cases = [(0, chunk, o0, o1, *r) for chunk, o0, o1, r in itertools.product(CHUNKS, offsets, offsets, REGIONS)]
    want = [e <= chunk and o0 + 64 <= o1 and chunk + o1 <= e + size for _, chunk, o0, o1, e, size in cases]
    assert inside(cases) == want and any(want)
    # a start past the region whose end, 64 bytes on, comes out small in 32 bits
    assert inside([(0, 4096, (1 << 32) - 16, 64, 4096, 8192)]) == [False]
    # a chunk so far behind the region that its place comes out in front of it in 64 bits
    assert inside([(0, (1 << 64) - 16, 0, 4200, 4096, 8192)]) == [False]


def test_raw_streams(inside):
    firsts = [0, 512, 4096, 8128, 8192, 1 << 32, ((1 << 32) - 512) * 65536]
    sizes = [16, 64, 512, 4096, 8192, (1 << 32) - 16]
    cases = [(1, chunk, first, n, *r) for chunk, first, n, r in itertools.product(CHUNKS, firsts, sizes, REGIONS)]
    want = [e <= chunk and chunk + first + n <= e + size for _, chunk, first, n, e, size in cases]
    assert inside(cases) == want and any(want)
