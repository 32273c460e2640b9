"""The decode kernels of the built library keep to the registers that the waves of zipmoe_kinds.h leave them, and use no scratch memory: read from the
metadata that the compiler puts beside the code."""
import os
import re
import struct
import subprocess

import msgpack
import pytest

from paper_2601_21198_amd.build import LIB_PATH

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
KINDS = ["short", "sparse", "fitting", "many", "mixed", "deep"]
WAVES = r"""
#include <cstdio>
#include "zipmoe_kinds.h"
using namespace zipmoe;
int main()
{
    for (int l = 0; l < 2; ++l)
        for (int k = kShortStreams; k <= kDeep; ++k) std::printf("%d %d\n", most_waves(static_cast<Kind>(k), l), bundle_waves(static_cast<Kind>(k), l));
}
"""
KERNEL = re.compile(r"zm_decode(?:_few)?_kernelILb([01])ELi(\d)ELN6zipmoe6StoresE\dELNS\w*_4KindE(\d)ELi(\d)E")


def kernels(path):
    """the metadata of every kernel in the library's code objects"""
    data, at, found = open(path, "rb").read(), 0, []
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    while (at := data.find(magic, at)) >= 0:
        pos, = struct.unpack_from("<Q", data, at + 24)
        entry = at + 32
        for _ in range(pos):
            offset, size, name = struct.unpack_from("<QQQ", data, entry)
            triple = data[entry + 24: entry + 24 + name]
            entry += 24 + name
            if b"gfx950" in triple:
                found += notes(data[at + offset: at + offset + size])
        at += 1
    return found


def notes(elf):
    table, entry, count = struct.unpack_from("<Q", elf, 40)[0], *struct.unpack_from("<HH", elf, 58)
    for i in range(count):
        kind, offset, size = (struct.unpack_from(f, elf, table + i * entry + o)[0] for f, o in (("<I", 4), ("<Q", 24), ("<Q", 32)))
        at = offset
        while kind == 7 and at < offset + size:                     # SHT_NOTE
            n, d, t = struct.unpack_from("<III", elf, at)
            body = at + 12 + (n + 3) // 4 * 4
            if t == 32:                                             # the kernels' metadata
                return msgpack.unpackb(elf[body: body + d])["amdhsa.kernels"]
            at = body + (d + 3) // 4 * 4
    return []


@pytest.fixture(scope="module")
def decode_kernels():
    found = {}
    for k in kernels(LIB_PATH):
        m = KERNEL.search(k[".name"])
        if m:
            found[k[".name"]] = tuple(int(x) for x in m.groups()) + (k,)
    return list(found.values())


@pytest.fixture(scope="module")
def waves(tmp_path_factory):
    at = tmp_path_factory.mktemp("waves")
    (at / "waves.cpp").write_text(WAVES)
    subprocess.check_call(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2601_21198_amd", "csrc"), str(at / "waves.cpp"), "-o", str(at / "waves")])
    rows = [tuple(int(x) for x in line.split()) for line in subprocess.check_output([str(at / "waves")], text=True).splitlines()]
    return {(long_codes, kind): rows[6 * long_codes + kind] for long_codes in (0, 1) for kind in range(6)}


def test_every_kernel_finds_its_waves(decode_kernels, waves):
    assert len(decode_kernels) > 100
    for long_codes, _, kind, bundle, k in decode_kernels:
        n = waves[long_codes, kind][bundle > 1]
        if KINDS[kind] == "sparse":
            n = 1 if long_codes else 3                              # its launches have no more
        registers = 512 // n // 8 * 8                               # of a SIMD's 512 a lane, by eights
        assert k[".vgpr_count"] <= registers, (k[".name"], k[".vgpr_count"], n)


def test_no_kernel_uses_scratch_memory(decode_kernels):
    for *_, k in decode_kernels:
        assert k[".private_segment_fixed_size"] == 0 and k[".vgpr_spill_count"] == 0 and k[".sgpr_spill_count"] == 0, k[".name"]
